"""Autotuner for the launch configuration of mixed-precision batches.

For each dividend width class of mp_divrem_ragged (<= 1024, 2048, 4096, 8192
limbs) it times a one-class batch of seeded random divisions under every
valid (threads per workgroup, hence limbs per thread in the linear passes;
persistent workgroups per compute unit) and installs the fastest with
mp_ragged_config.  Then it times the two process-wide knobs, each on the calls
that read it: how long the blocks of quotient limbs are (MP_KNOB_SMALL_LIMIT,
in limbs of the inverse's last Newton step) on a seeded mixed batch, and from
which operand length mp_mul_batch moves from the vector ALU to the matrix cores
(MP_KNOB_MFMA_MIN) on products with short operands of the lengths in question;
and installs the fastest of each.  Results are cached in a JSON file keyed by
the device (architecture name and compute-unit count) and by a hash of the
kernel sources and of this file, so a cache entry is never applied to a
different chip, to changed kernels or if it was chosen another way.  Timing runs on the GPU; nothing here computes any part of
a division, and every setting gives the same bits.
"""
import hashlib
import json
import os
import time

import numpy as np

from . import inputs as I

CLASS_WIDTHS = (1024, 2048, 4096, 8192)
THREADS = (256, 512, 1024)
WGS_PER_CU = (1, 2, 3, 4, 6, 8)
DEFAULT_CACHE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "tuned_ragged.json")
_CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "csrc")


def source_hash():
    h = hashlib.sha256()
    for f in [os.path.join(_CSRC, f) for f in sorted(os.listdir(_CSRC))] + [os.path.abspath(__file__)]:
        with open(f, "rb") as fh:
            h.update(os.path.basename(f).encode() + b"\0" + fh.read())
    return h.hexdigest()[:16]


def device_key():
    import torch
    p = torch.cuda.get_device_properties(torch.cuda.current_device())
    return "%s/%dcu/%s" % (p.gcnArchName.split(":")[0], p.multi_processor_count, source_hash())


def candidates(cls):
    w = CLASS_WIDTHS[cls]
    return [(t, g) for t in THREADS if 8 * t >= w for g in WGS_PER_CU]


def class_batch(cls, count):
    """Seeded one-class divisions: width n of the class, divisor length
    uniform in [ceil(n/4), n] (the mixed workload's distribution)."""
    n = CLASS_WIDTHS[cls]
    st = I.instance_states(I.SEED_C4 ^ (0x7E0000 + cls), np.arange(count))
    nvs = I.uniform_int(I.substream(st, 2), (n + 3) // 4, n)
    s0, s1 = I.substream(st, 0), I.substream(st, 1)
    us = list(I.limbs_top_nonzero(s0, n))
    vs = [I.limbs_top_nonzero(s1[r:r + 1], int(nv))[0] for r, nv in enumerate(nvs)]
    return us, vs


def _time(call, reps):
    import torch
    call()
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(reps):
        call()
    e1.record()
    torch.cuda.synchronize()
    return e0.elapsed_time(e1) / reps


AUTO = -2           # the library's own limit (MP_SMALL_LIMIT_AUTO)
SMALL_LIMITS = (AUTO, 32, 48, 64, 80, 96, 112, 128, 136)
MFMA_MINS = (32, 64, 96, 128)
MFMA_MIN_DEFAULT = 64
AUTO_SLACK = 1.01    # the library's own settings are kept unless another is >1% faster


def product_calls(batch=2048, hi=1024):
    """Products whose short operand lies between two of MFMA_MINS, one call for each gap."""
    import torch
    from . import binding
    gen = torch.Generator(device="cuda")
    gen.manual_seed(I.SEED_C4)
    limbs = lambda n: torch.randint(-2 ** 31, 2 ** 31, (batch, n), dtype=torch.int32, device="cuda", generator=gen)
    pairs = [(limbs((a + b) // 2), limbs(hi)) for a, b in zip(MFMA_MINS, MFMA_MINS[1:])]
    return [lambda a=a, b=b: binding.mul(a, b) for a, b in pairs]


ROUNDS = 3          # over all values in turn
WARM_S = 0.06       # before them: from idle the clock rises for some 25 ms


def _tune_knob(knob, name, values, default, time_ms, log=None):
    """Set the knob to the value of the shortest time, or to the default where that is
    within AUTO_SLACK of it; returns (value, ms)."""
    from . import binding
    start = time.perf_counter()
    while time.perf_counter() - start < WARM_S:
        time_ms()
    best = dict.fromkeys(values, float("inf"))
    for _ in range(ROUNDS):
        for x in values:
            binding.set_knob(knob, x)
            best[x] = min(best[x], time_ms())
    if log:
        for x, ms in best.items():
            log("knob %s %s: %.3f ms" % (name, "auto" if x == AUTO else x, ms))
    x = min(values, key=best.get)
    x = default if best[default] <= best[x] * AUTO_SLACK else x
    binding.set_knob(knob, x)
    return x, best[x]


def tune_knobs(count=1024, reps=3, log=None):
    """Time every small_limit on a seeded mixed batch (all four width classes) and
    every mfma_min on products (divisions do not read it); installs the fastest of
    each and returns them as {knob: value, 'ms': ms of the mixed batch}."""
    from . import binding, ragged
    m = I.config_c4(index=np.arange(0, 8 * count, 8))
    rb = binding.Ragged(ragged.pack(m["u"], m["v"]))
    sl, ms = _tune_knob(binding.MP_KNOB_SMALL_LIMIT, "small_limit", SMALL_LIMITS, AUTO, lambda: _time(rb.run, reps), log)
    calls = product_calls()
    mm, _ = _tune_knob(binding.MP_KNOB_MFMA_MIN, "mfma_min", MFMA_MINS, MFMA_MIN_DEFAULT,
                       lambda: sum(_time(f, 10 * reps) for f in calls), log)
    return {"small_limit": sl, "mfma_min": mm, "ms": ms}


def smallest_classed_batch():
    """Instances from which mp_divrem_ragged runs its class kernels: up to two per
    compute unit take one launch that reads no class configuration."""
    import torch
    return 2 * torch.cuda.get_device_properties(torch.cuda.current_device()).multi_processor_count + 1


def tune(counts=(2048, 1024, 1024, 768), reps=3, log=None):
    """Time every candidate per class on a batch of `counts` instances (at least
    as many as reach the class kernels); returns {cls: (threads, wgs_per_cu, ms)}."""
    from . import binding, ragged
    best, least = {}, smallest_classed_batch()
    for cls in range(len(CLASS_WIDTHS)):
        us, vs = class_batch(cls, max(counts[cls], least))
        rb = binding.Ragged(ragged.pack(us, vs))
        times = []
        for t, g in candidates(cls):
            binding.ragged_config(cls, t, g)
            ms = _time(rb.run, reps)
            times.append((ms, t, g))
            if log:
                log("class %d (<= %d limbs): threads %d, %d WG/CU: %.3f ms" % (cls, CLASS_WIDTHS[cls], t, g, ms))
        ms, t, g = min(times)
        binding.ragged_config(cls, t, g)
        best[cls] = (t, g, ms)
    return best


def apply(entry):
    """Install a cache entry: {'classes': {cls: (threads, wgs_per_cu, ms)},
    'knobs': {'small_limit': .., 'mfma_min': ..}}."""
    from . import binding
    for cls, (t, g, _) in entry["classes"].items():
        binding.ragged_config(int(cls), int(t), int(g))
    kn = entry.get("knobs")
    if kn:
        binding.set_knob(binding.MP_KNOB_SMALL_LIMIT, int(kn["small_limit"]))
        binding.set_knob(binding.MP_KNOB_MFMA_MIN, int(kn["mfma_min"]))


def ensure(cache=DEFAULT_CACHE, log=None):
    """Install the cached configuration for this device, tuning (and writing
    the cache, where writable) when there is none."""
    key = device_key()
    data = {}
    if os.path.exists(cache):
        with open(cache) as fh:
            data = json.load(fh)
    if key in data and "classes" in data[key]:
        apply(data[key])
        return data[key], False
    best = tune(log=log)
    knobs = tune_knobs(log=log)
    data[key] = {"classes": {str(k): list(v) for k, v in best.items()}, "knobs": knobs}
    try:
        with open(cache, "w") as fh:
            json.dump(data, fh, indent=1, sort_keys=True)
    except OSError:
        pass
    return data[key], True
