"""Few rows times a wide row-major B: the leaf that turns B's blocks on their way through LDS,
at the edges of its tiles and stages, against the oracle."""
import numpy as np
import pytest

import bmmgen
import oracle
from gpu_util import announce, empty_dev, from_dev, to_dev, words

pytestmark = pytest.mark.gpu

# one and two rows of tiles; 192 to 256 tiles, 448 to 512 and more, whole and ragged, the last
# tile one word or less; k: a bit, part of a word, of a stage, whole stages, 1 to 6; the last
# three are just outside of what this leaf takes
SHAPES = [(129, 1, 24449), (256, 64, 32768), (255, 512, 57217), (129, 513, 57345),
          (200, 1000, 65536), (400, 1024, 12290), (512, 1537, 16384), (385, 2113, 28740),
          (256, 3072, 57600), (128, 600, 65536), (256, 600, 32769), (384, 600, 16384)]


@pytest.fixture(scope="module")
def bmm():
    import paper_1909_01554_amd as bmm
    return bmm


@pytest.mark.parametrize("m,k,n", SHAPES)
@pytest.mark.parametrize("leaf", [2, 3])
@pytest.mark.parametrize("sr", [oracle.GF2, oracle.BOOLEAN])
def test_few_rows(bmm, m, k, n, leaf, sr):
    import torch
    dist = bmmgen.Dist.half()
    A = bmmgen.fill_cpu(m, k, 31, bmmgen.TAG_A, dist)
    if sr == oracle.BOOLEAN:  # sparse: about two ones a row
        rng = np.random.default_rng(k)
        A = np.zeros_like(A)
        for j in rng.integers(0, k, 2):
            A[:, j // 64] |= np.uint64(1 << int(j % 64))
    B = bmmgen.fill_cpu(k, n, 31, bmmgen.TAG_B, dist)
    want = oracle.mul(A, B, k, n, sr)
    ldb, ldc = words(n) + 1, words(n) + 3
    C = empty_dev(m, ldc, fill=-1)
    mul = bmm.bmm_gf2 if sr == oracle.GF2 else bmm.bmm_boolean
    announce("few rows", m, k, n, leaf, sr)
    mul(to_dev(A), to_dev(B, ldb), C, m, k, n, options=bmm.Options(leaf=leaf))
    torch.cuda.synchronize()
    got = C.cpu().numpy().view(np.uint64)
    assert np.array_equal(got[:, :words(n)], want)
    assert (got[:, words(n):] == np.uint64(2**64 - 1)).all()
    # accumulating: the same product again clears it (GF(2)) or leaves it (OR)
    mul(to_dev(A), to_dev(B, ldb), C, m, k, n, options=bmm.Options(leaf=leaf), accumulate=True)
    torch.cuda.synchronize()
    got = C.cpu().numpy().view(np.uint64)
    assert np.array_equal(got[:, :words(n)], want if sr == oracle.BOOLEAN else want ^ want)
