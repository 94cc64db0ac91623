"""The default rule between small and large tiles of the matrix-core leaves, at its lines (host
logic only; results do not depend on it)."""
import pytest


@pytest.fixture
def bmm():
    import paper_1909_01554_amd as bmm
    bmm.bmm_finalize()
    return bmm


# sizes, and whether int8 and fp4 take the small tiles
@pytest.mark.parametrize("m,k,n,i8,f4", [
    (4342, 256, 1831, True, True),       # 272 wide or 255 tall workgroups, 510 small ones
    (4342, 8192, 1831, True, True),
    (40000, 4096, 128, True, True),      # wide ones would be half empty
    (1000, 257, 6000, True, False),      # 192 wide, 376 small; 1504 of 64 x 64 from registers
    (1000, 256, 6000, True, True),       # while k is short
    (1000, 321, 6000, False, False),
    (4096, 64, 4096, False, False),      # 4096 of 64 x 64
    (64, 2047, 200000, True, True),      # one row of tiles
    (200000, 5000, 64, True, True),
    (7872, 512, 2944, False, False),     # 744 and 1426
    (5000, 512, 5000, True, False),      # 800 and 1600: fp4 by its short k
    (5000, 513, 5000, True, True),
    (5001, 7003, 3333, True, True),
    (4096, 4096, 4096, False, False),
    (1000, 256, 1000, True, True),       # up to 512 of 64 x 64
])
def test_small_tiles(bmm, m, k, n, i8, f4):
    for leaf, small in ((bmm.LEAF_MFMA_I8, i8), (bmm.LEAF_MFMA_F4, f4)):
        tile = bmm.bmm_leaf_choice(bmm.GF2, m, k, n, options=bmm.Options(leaf=leaf))[1]
        assert (tile == 2) == small, (leaf, tile)
