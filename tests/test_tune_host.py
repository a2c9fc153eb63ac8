"""What the tuner chooses from which times, without a GPU (stand-in batches and times)."""
import pytest

from paper_2606_06386_amd import binding, tune


class Batch:
    def __init__(self, packed, device="cuda"):
        self.count = len(packed["desc"])

    def run(self):
        pass


@pytest.fixture
def host(monkeypatch):
    """the tuner over stand-in batches, knobs and configurations put back afterwards"""
    old = [binding.get_knob(k) for k in (binding.MP_KNOB_MFMA_MIN, binding.MP_KNOB_SMALL_LIMIT)]
    monkeypatch.setattr(binding, "Ragged", Batch)
    yield monkeypatch
    for k, x in zip((binding.MP_KNOB_MFMA_MIN, binding.MP_KNOB_SMALL_LIMIT), old):
        binding.set_knob(k, x)


@pytest.mark.parametrize("product_ms,chosen", [
    ({32: 1.2, 64: 1.1, 96: 1.0, 128: 1.3}, 96), ({32: 1.2, 64: 1.005, 96: 1.0, 128: 1.3}, 64),
    ({32: 0.9, 64: 1.0, 96: 1.1, 128: 1.3}, 32)])
def test_mfma_min_is_chosen_by_products(host, product_ms, chosen):
    """Divisions do not read mfma_min: differences between their times are noise."""
    def time(call, reps):
        mm = binding.get_knob(binding.MP_KNOB_MFMA_MIN)
        if isinstance(getattr(call, "__self__", call), Batch):
            return 1.0 - mm / 1e5 + (0.5 if binding.get_knob(binding.MP_KNOB_SMALL_LIMIT) > 0 else 0.0)
        return product_ms[mm]
    host.setattr(tune, "_time", time)
    host.setattr(tune, "product_calls", lambda: [lambda: None], raising=False)
    got = tune.tune_knobs(count=4)
    assert got["mfma_min"] == chosen == binding.get_knob(binding.MP_KNOB_MFMA_MIN)
    assert got["small_limit"] == tune.AUTO == binding.get_knob(binding.MP_KNOB_SMALL_LIMIT)


def test_small_limit_clearly_faster_than_the_librarys_own(host):
    host.setattr(tune, "_time", lambda call, reps: 0.9 if binding.get_knob(binding.MP_KNOB_SMALL_LIMIT) == 96 else 1.0)
    host.setattr(tune, "product_calls", lambda: [lambda: None], raising=False)
    assert tune.tune_knobs(count=4)["small_limit"] == 96 == binding.get_knob(binding.MP_KNOB_SMALL_LIMIT)


def test_class_configurations_are_timed_where_they_are_read(host):
    """Batches of at most two instances per compute unit run outside the classes."""
    seen = {}
    host.setattr(tune, "class_batch", lambda cls, count: seen.setdefault(cls, count) and ([[1]], [[1]]))
    host.setattr(tune, "_time", lambda call, reps: 1.0)
    host.setattr(tune, "smallest_classed_batch", lambda: 513, raising=False)
    host.setattr(binding, "ragged_config", lambda cls, threads, wgs: None)
    best = tune.tune(counts=(32, 16, 600, 4), reps=1)
    assert set(best) == {0, 1, 2, 3} and seen == {0: 513, 1: 513, 2: 600, 3: 513}
