"""Products on the engine that the default cut-over does not give them: short
operands on the matrix cores, long ones on the vector ALU, against the oracle
(odd widths, runs of zeros and ones, every workgroup size)."""
import numpy as np
import pytest

import oracle
from test_gpu_mul_shapes import _operands

pytestmark = pytest.mark.gpu


@pytest.fixture
def mp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2606_06386_amd import binding
    binding.lib()
    old = binding.get_knob(binding.MP_KNOB_MFMA_MIN)
    yield binding
    binding.set_knob(binding.MP_KNOB_MFMA_MIN, old)


def _check(mp, na, nb, batch):
    import torch
    a, b = _operands(np.random.default_rng(na * 8191 + nb), na, nb)
    dev = lambda x: torch.from_numpy(x.view(np.int32)).cuda()  # noqa: E731
    rep = -(-batch // 8)
    want = torch.from_numpy(oracle.mul(a, b).view(np.int32)).cuda().repeat(rep, 1)[:batch]
    c = mp.mul(dev(a).repeat(rep, 1)[:batch].contiguous(), dev(b).repeat(rep, 1)[:batch].contiguous())
    bad = torch.nonzero((c != want).any(dim=1)).flatten().tolist()
    assert not bad, f"{na} x {nb}, batch {batch}: products {[j % 8 for j in bad[:8]]} differ"


# long operands for one to eight strips, and for each size of the groups of four (from 6144 strips, or 17 a product)
@pytest.mark.parametrize("lo", [1, 2, 3, 7, 8, 16, 31, 32, 33, 48, 63])
def test_short_operands_on_the_matrix_cores(mp, lo):
    mp.set_knob(mp.MP_KNOB_MFMA_MIN, 1)
    for hi, batch in ((lo, 8), (lo + 1, 8), (64, 8), (257, 9), (1025, 8), (1700, 8), (1900, 900), (2049, 8), (3001, 700),
                      (4100, 8), (8100, 8), (8192, 8)):
        _check(mp, lo, hi, batch)
        _check(mp, hi, lo, batch)


@pytest.mark.parametrize("na,nb,batch", [
    (64, 64, 8), (65, 300, 9), (255, 257, 8), (333, 1531, 600), (1000, 1001, 8), (2048, 2048, 8), (2049, 2049, 8),
    (4096, 4096, 8), (4096, 4099, 8), (8192, 1, 8), (8192, 1015, 8), (8191, 8190, 8), (8192, 8192, 8)])
def test_long_operands_on_the_vector_alu(mp, na, nb, batch):
    mp.set_knob(mp.MP_KNOB_MFMA_MIN, 1 << 30)
    _check(mp, na, nb, batch)
