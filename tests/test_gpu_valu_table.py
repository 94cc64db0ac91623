"""The VALU leaf's table form (large cubic products), bit-exact: one workgroup round of 1024 x
1024 tiles with ragged last ones, k from one bit over the 16 rows of a phase and the 128 of a
quad to past them, B row-major and transposed, odd pitches, fresh and accumulated."""
import numpy as np
import pytest

import bmmgen
import oracle
from gpu_util import announce, empty_dev, from_dev, to_dev, words

pytestmark = pytest.mark.gpu

SEMIRINGS = [("gf2", oracle.GF2), ("bool", oracle.BOOLEAN)]


@pytest.fixture(scope="module")
def bmm():
    import paper_1909_01554_amd as bmm
    return bmm


@pytest.mark.parametrize("sname,sr", SEMIRINGS)
@pytest.mark.parametrize("m,k,n", [(12700, 1, 12700), (11000, 16, 14593), (14593, 17, 11001),
                                   (12700, 127, 12673), (12800, 128, 12800), (12700, 145, 12700),
                                   (11000, 300, 14656)])
def test_table_form(bmm, sname, sr, m, k, n):
    p = bmmgen.Dist.half() if sr == oracle.GF2 else bmmgen.Dist.inv_sqrt(k)
    A = bmmgen.fill_cpu(m, k, 7 + k, bmmgen.TAG_A, p)
    B = bmmgen.fill_cpu(k, n, 7 + k, bmmgen.TAG_B, p)
    want = oracle.mul(A, B, k, n, sr)
    assert bmm.bmm_leaf_choice(sr, m, k, n, options=bmm.Options(leaf=1)) == (1, 2)
    fn = bmm.bmm_gf2 if sr == oracle.GF2 else bmm.bmm_boolean
    for pad in (0, 1):
        announce("valu table", sname, (m, k, n), pad)
        Cd = empty_dev(m, words(n) + pad, fill=-1)
        fn(to_dev(A, A.shape[1] + pad), to_dev(B, B.shape[1] + pad), Cd, m, k, n,
           options=bmm.Options(leaf=1))
        got = from_dev(Cd)
        assert np.array_equal(got[:, :words(n)], want)
        assert pad == 0 or (got[:, -1] == np.uint64(2**64 - 1)).all()
    C0 = bmmgen.fill_cpu(m, n, 7 + k, 0xC0, bmmgen.Dist.half())
    BT = to_dev(np.zeros((n, words(k)), dtype=np.uint64))
    bmm.bmm_transpose(to_dev(B), BT, k, n)
    announce("valu table, B transposed, accumulated", sname, (m, k, n))
    Cd = to_dev(C0)
    fn(to_dev(A), BT, Cd, m, k, n, options=bmm.Options(leaf=1), b_transposed=True, accumulate=True)
    assert np.array_equal(from_dev(Cd), (want ^ C0) if sr == oracle.GF2 else (want | C0))
