"""Products in every split of strips over waves, against the oracle.

A product's columns are dealt to waves in strips of 256, one, two, four or
twice four per wave by its size and the batch; a wave's carries stay in
registers and pass to the next wave's columns, through whole groups of strips
where the limbs are all ones or zeros.  Sizes on both sides of each rule, odd
widths (unaligned output rows), and operands whose products are runs of zeros
and ones, bit-exact."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2606_06386_amd import binding
    binding.lib()
    return binding


def _operands(rng, na, nb):
    """random; all ones times all ones, one, B^k and a sparse number; borrows and carries through long runs"""
    a = rng.integers(0, 2 ** 32, (8, na), dtype=np.uint64).astype(np.uint32)
    b = rng.integers(0, 2 ** 32, (8, nb), dtype=np.uint64).astype(np.uint32)
    a[1], b[1] = 0xFFFFFFFF, 0xFFFFFFFF
    a[2], b[2] = 0xFFFFFFFF, 0
    b[2, 0] = 1
    a[3], b[3] = 0xFFFFFFFF, 0
    b[3, nb - 1] = 0x80000000
    a[4], b[4] = 0, 0
    a[4, ::256], b[4, 0], b[4, nb - 1] = 1, 0xFFFFFFFF, 1
    a[5], b[5] = 0x7F7F7F7F, 0x80808080
    a[6, na // 3:] = 0
    b[7] = 0
    return a, b


# (na, nb, batch): the smallest batches of a rule's two sides
@pytest.mark.parametrize("na,nb,batch", [
    (64, 64, 8), (700, 324, 8), (769, 767, 8), (769, 768, 8), (769, 768, 900), (1024, 1024, 800), (1015, 1033, 800),
    (1016, 1033, 300), (2047, 2049, 400), (2048, 2048, 1040), (1016, 2100, 1300), (1015, 3000, 500), (2050, 2047, 8),
    (4000, 4192, 8), (4096, 4095, 270), (4097, 4096, 8), (8192, 1015, 8), (8191, 2001, 8), (8192, 2000, 420),
    (8192, 8192, 8), (8192, 8192, 260)])
def test_mul_shapes(mp, na, nb, batch):
    import torch
    a, b = _operands(np.random.default_rng(na * 8191 + nb), na, nb)
    dev = lambda x: torch.from_numpy(x.view(np.int32)).cuda()  # noqa: E731
    rep = -(-batch // 8)
    c = mp.mul(dev(a).repeat(rep, 1)[:batch].contiguous(), dev(b).repeat(rep, 1)[:batch].contiguous())
    want = torch.from_numpy(oracle.mul(a, b).view(np.int32)).cuda().repeat(rep, 1)[:batch]
    bad = torch.nonzero((c != want).any(dim=1)).flatten().tolist()
    assert not bad, f"{na} x {nb}, batch {batch}: products {[j % 8 for j in bad[:8]]} differ (instances {bad[:8]})"
