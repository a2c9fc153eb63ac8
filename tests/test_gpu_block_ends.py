"""Quotients of whole numbers of blocks of 252 limbs and of one or two limbs more
or less (up to five blocks), with divisors of one to three strips, in batches
of every kind of kernel."""
import random

import pytest

import test_gpu_blocks as blocks
import test_gpu_division_modes as modes

pytestmark = pytest.mark.gpu
ENDS = [252 * n + i for n in (1, 2, 3, 4, 5) for i in (-1, 0, 1, 2)]


@pytest.mark.parametrize("d", ENDS)
def test_quotients_at_the_ends_of_blocks(d):
    from paper_2606_06386_amd import binding
    rng = random.Random(d)
    for k in (1, 62, 247, 255, 510, 700):
        c = blocks._cases(rng, d, k)
        blocks._check(binding, blocks._stack([u for u, _ in c], d + k), blocks._stack([v for _, v in c], k + 1), d,
                      f"d={d} k={k}")


@pytest.mark.parametrize("d,k", [(756, 254), (757, 510), (1008, 255), (1009, 700)])
@pytest.mark.parametrize("per_cu", [0, 3, 4, 5])
def test_ends_of_blocks_in_every_kind_of_batch(d, k, per_cu):
    modes.test_every_kind_of_batch(d, k, per_cu)
