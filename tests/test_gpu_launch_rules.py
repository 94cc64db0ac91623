"""Products at the lines of the launch rules, bit-exact against the oracle."""
import numpy as np
import pytest

import bmmgen
import oracle
from gpu_util import announce, empty_dev, from_dev, to_dev, words

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bmm():
    import paper_1909_01554_amd as bmm
    yield bmm
    bmm.bmm_debug_fail_allocations(0)
    bmm.bmm_finalize()


def operands(m, k, n, sr, seed):
    dist = bmmgen.Dist.half() if sr == oracle.GF2 else bmmgen.Dist.inv_sqrt(k)
    A = bmmgen.fill_cpu(m, k, seed, bmmgen.TAG_A, dist)
    B = bmmgen.fill_cpu(k, n, seed, bmmgen.TAG_B, dist)
    return A, B


def product(bmm, sr):
    return bmm.bmm_gf2 if sr == oracle.GF2 else bmm.bmm_boolean


@pytest.mark.parametrize("leaf", [2, 3])
@pytest.mark.parametrize("sr", [oracle.GF2, oracle.BOOLEAN])
@pytest.mark.parametrize("k", [3311, 3312])  # 23 x 24 tiles of 64 x 64: split from 6 bits each
def test_tile_4_past_two_workgroups_per_cu(bmm, k, sr, leaf):
    m, n = 1472, 1473
    A, B = operands(m, k, n, sr, 5)
    C = empty_dev(m, words(n) + 1, fill=-1)
    announce("tile 4", m, k, n, sr, leaf)
    product(bmm, sr)(to_dev(A), to_dev(B), C, m, k, n, options=bmm.Options(leaf=leaf, tile=4))
    got = from_dev(C)
    assert np.array_equal(got[:, :words(n)], oracle.mul(A, B, k, n, sr))
    assert (got[:, -1] == np.uint64(2**64 - 1)).all()
