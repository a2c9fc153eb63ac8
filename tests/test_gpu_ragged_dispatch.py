"""Ragged batches on both sides of the sizes where their launches change.

Batches of at most two instances per compute unit run as one launch with a
workgroup per instance; larger ones are bucketed into width classes, the widest
of which runs one or two workgroups per compute unit.  Every width class,
broken descriptors among the instances, both entry points, captured and eager;
operands with zero top limbs, checked against Python's integers."""
import random

import numpy as np
import pytest

from paper_2606_06386_amd import ragged as R

pytestmark = pytest.mark.gpu
WIDTHS = (1024, 2048, 4096, 8192)
CANARY = 0x5A5A5A5A


def _limbs(x, n):
    return np.frombuffer(x.to_bytes(4 * n, "little"), dtype="<u4").astype(np.uint32)


def _batch(count, widths=WIDTHS):
    rng = random.Random(count)
    us, vs, want = [], [], []
    for j in range(count):
        n = widths[j % len(widths)] - rng.choice((0, 1, 500))
        k, d = rng.randint(1, 60), rng.randint(1, 40) if j % 31 else rng.randint(200, 450)
        m = rng.randint(k, n)
        u = rng.getrandbits(32 * (k + d))
        v = rng.getrandbits(32 * k) if j % 17 else 0
        q, r = divmod(u, v) if v else (0, 0)
        us.append(_limbs(u, n))
        vs.append(_limbs(v, m))
        want.append((q, r, 0 if v else 1))
    return us, vs, want


@pytest.mark.parametrize("per_cu", [1.0, 2.0, 6.0])
@pytest.mark.parametrize("extra", [0, 4])
@pytest.mark.parametrize("entry", ["run", "run_static"])
def test_ragged_both_sides_of_each_launch_rule(per_cu, extra, entry):
    import torch
    from paper_2606_06386_amd import binding
    count = int(per_cu * torch.cuda.get_device_properties(0).multi_processor_count) + extra
    us, vs, want = _batch(count)
    packed = R.pack(us, vs)
    d = packed["desc"]
    broken = {0: 4, count // 2: 4, count - 1: 4}
    d["u_off"][0] = len(packed["u_pool"]) - d["nu"][0] + 1
    d["nv"][count // 2] = 8193
    d["r_off"][count - 1] = packed["r_limbs"] - d["nv"][count - 1] + 1
    rb = binding.Ragged(packed)
    s, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()

    def check(label):
        torch.cuda.synchronize()
        q, r, st = (x.cpu().numpy().view(np.uint32) for x in (rb.q, rb.r, rb.status))
        bad = []
        for j in range(count):
            x = d[j]
            qj = q[x["q_off"]:x["q_off"] + x["nq"]]
            if j in broken:
                ok = st[j] == 4 and (qj == CANARY).all()
            else:
                rj = r[x["r_off"]:x["r_off"] + x["nv"]]
                ok = st[j] == want[j][2] and (qj == _limbs(want[j][0], len(qj))).all() and (
                    rj == _limbs(want[j][1], len(rj))).all()
            if not ok:
                bad.append(j)
        assert not bad, f"{label}: {len(bad)} of {count}, first {bad[:8]}, status {st[bad[:8]]}"
        rb.q.fill_(CANARY)
        rb.r.fill_(CANARY)
        rb.status.fill_(-1)

    rb.q.fill_(CANARY)
    getattr(rb, entry)()
    check("eager")
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        getattr(rb, entry)()
        s.synchronize()
        with torch.cuda.graph(g, stream=s):
            getattr(rb, entry)()
    torch.cuda.synchronize()
    check("before the replays")
    for rep in range(3):
        torch.arange(1 << 16, device="cuda").sum().item()      # unrelated eager work
        g.replay()
        check(f"replay {rep}")


@pytest.mark.parametrize("widths", [(8192,), (4096, 8192, 8192, 8192)])
def test_ragged_batches_of_the_widest_class(widths):
    """(with no or few instances of the next class beside)"""
    import torch
    from paper_2606_06386_amd import binding
    us, vs, want = _batch(800, widths)
    packed = R.pack(us, vs)
    rb = binding.Ragged(packed)
    rb.run()
    torch.cuda.synchronize()
    q, r, st = (x.cpu().numpy().view(np.uint32) for x in (rb.q, rb.r, rb.status))
    qs, rs = R.unpack(q, packed["desc"], "q"), R.unpack(r, packed["desc"], "r")
    bad = [j for j in range(800) if st[j] != want[j][2] or (qs[j] != _limbs(want[j][0], len(qs[j]))).any()
           or (rs[j] != _limbs(want[j][1], len(rs[j]))).any()]
    assert not bad, f"{len(bad)} mismatching instances, first {bad[:8]}"
