"""In-place basis changes with the lean levels, whose operands have to be in the alternative
basis: the caller's operands are changed, and hold their own words again afterwards."""
import numpy as np
import pytest

import bmmgen
import oracle
from gpu_util import announce, empty_dev, from_dev, to_dev, words

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bmm():
    import paper_1909_01554_amd as bmm
    return bmm


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("depth,ds", [(1, 1), (3, 2), (4, 2)])
@pytest.mark.parametrize("b_t", [False, True])
@pytest.mark.parametrize("scheme", [0, 1, 2])
@pytest.mark.parametrize("leaf", [2, 3])
def test_lean_levels_in_place(bmm, scheme, b_t, depth, ds, accumulate, leaf):
    import torch
    from oracle import brute
    m, k, n = 512, 1024, 2048
    seed = 600 + 10 * depth + scheme + (5 if b_t else 0)
    A = bmmgen.fill_cpu(m, k, seed, bmmgen.TAG_A, bmmgen.Dist.half())
    B = bmmgen.fill_cpu(k, n, seed, bmmgen.TAG_B, bmmgen.Dist.half())
    C0 = bmmgen.fill_cpu(m, n, seed, 0xC, bmmgen.Dist.half())
    Bin = brute.pack(brute.unpack(B, n).T.copy()) if b_t else B
    opts = bmm.Options(leaf=leaf, depth_serial=ds, depth_parallel=depth - ds, scheme=scheme,
                       flags=bmm.FLAG_LEAN_WORKSPACE)
    nbytes, _, _ = bmm.bmm_gf2_strassen_workspace(m, k, n, depth, opts, b_transposed=b_t,
                                                  inplace_basis=True)
    ws = torch.empty(nbytes // 8 + 1, dtype=torch.int64, device="cuda")
    Ad, Bd = to_dev(A, words(k) + 1), to_dev(Bin, Bin.shape[1] + 2)
    Cd = to_dev(C0) if accumulate else empty_dev(m, words(n), fill=-1)
    announce("strassen lean in place", scheme, b_t, depth, ds, accumulate, leaf)
    bmm.bmm_gf2_strassen(Ad, Bd, Cd, m, k, n, ws, depth=depth, options=opts, b_transposed=b_t,
                         accumulate=accumulate, inplace_basis=True)
    prod = oracle.mul(A, B, k, n, oracle.GF2)
    assert np.array_equal(from_dev(Cd), (C0 ^ prod) if accumulate else prod)
    assert np.array_equal(from_dev(Ad, words(k)), A)
    assert np.array_equal(from_dev(Bd, Bin.shape[1]), Bin)
