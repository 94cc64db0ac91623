"""The out-of-core host levels with A and B kept in HBM (each block uploaded once) and, when
there is no memory for that, through the staging slots: same product, bit for bit."""
import numpy as np
import pytest

import bmmgen
import oracle
from gpu_util import announce, words

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bmm():
    import paper_1909_01554_amd as bmm
    yield bmm
    bmm.bmm_debug_fail_allocations(0)


@pytest.mark.parametrize("scheme", [0, 1, 2])
@pytest.mark.parametrize("blk,dh", [(256, 1), (128, 2), (4096, 1)])
@pytest.mark.parametrize("resident", [True, False])
def test_host_levels_resident_and_staged(bmm, scheme, blk, dh, resident):
    import torch
    n = blk << dh
    A = bmmgen.fill_cpu(n, n, 41 + dh, bmmgen.TAG_A, bmmgen.Dist.half())
    B = bmmgen.fill_cpu(n, n, 41 + dh, bmmgen.TAG_B, bmmgen.Dist.half())
    pad = 3 if blk == 256 else 0  # host pitches beyond the rows

    def host(x):
        y = torch.full((n, words(n) + pad), -1, dtype=torch.int64)
        y[:, :words(n)] = torch.from_numpy(x.view(np.int64))
        return y.pin_memory()

    Ah, Bh = host(A), host(B)
    Ch = torch.full((n, words(n) + pad), -1, dtype=torch.int64).pin_memory()
    announce("ooc resident", scheme, blk, dh, resident)
    # the first allocation is A's place in HBM: without it the blocks are staged
    bmm.bmm_debug_fail_allocations(0 if resident else 1)
    bmm.bmm_ooc(oracle.GF2, Ah, Bh, Ch, n, n, n, block=blk, options=bmm.Options(scheme=scheme))
    bmm.bmm_debug_fail_allocations(0)
    got = Ch.numpy().view(np.uint64)
    assert np.array_equal(got[:, :words(n)], oracle.mul(A, B, n, n, oracle.GF2))
    assert pad == 0 or (got[:, words(n):] == np.uint64(2**64 - 1)).all()
    up, _, down, _ = bmm.bmm_ooc_last_transfers()
    assert down == A.nbytes
    assert up == 2 * A.nbytes if resident else up > 2 * A.nbytes
