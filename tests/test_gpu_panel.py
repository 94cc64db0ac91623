"""GPU parity of the LDS-staged matrix-core leaf (panel_tile.h) at the sizes where it can go
wrong: the edges of its 128 x 256 and 256 x 128 workgroup tiles, the remainders of a stage
(512 bits) and of a round (256 bits), rows of odd pitch, pitches past 32-bit row offsets,
and the longest k its counts hold.  All results are bit-exact."""
import numpy as np
import pytest

import bmmgen
import oracle
from gpu_util import announce, empty_dev, from_dev, to_dev, words

pytestmark = pytest.mark.gpu

SEMIRINGS = [("gf2", oracle.GF2), ("bool", oracle.BOOLEAN)]
FORMATS = [("int8", 2), ("fp4", 3)]


@pytest.fixture(scope="module")
def bmm():
    import paper_1909_01554_amd as bmm
    return bmm


def product(bmm, sr):
    return bmm.bmm_gf2 if sr == oracle.GF2 else bmm.bmm_boolean


# tile edges (128, 256 and one beyond, short of a word and past it) x stage and round edges
SHAPES = [(128, 512, 256), (129, 513, 257), (256, 511, 128), (257, 1024, 129), (1, 256, 320),
          (64, 257, 64), (300, 1025, 40), (127, 64, 255), (260, 1600, 520), (140, 2561, 600)]


@pytest.mark.parametrize("sname,sr", SEMIRINGS)
@pytest.mark.parametrize("fname,leaf", FORMATS)
@pytest.mark.parametrize("pad", [0, 1])
def test_tile_and_stage_edges(bmm, sname, sr, fname, leaf, pad):
    for i, (m, k, n) in enumerate(SHAPES):
        p = None if sr == oracle.GF2 else bmmgen.Dist.inv_sqrt(k)
        A = bmmgen.fill_cpu(m, k, 71 + i, bmmgen.TAG_A, p or bmmgen.Dist.half())
        B = bmmgen.fill_cpu(k, n, 71 + i, bmmgen.TAG_B, p or bmmgen.Dist.half())
        want = oracle.mul(A, B, k, n, sr)
        announce("panel", sname, fname, (m, k, n), pad)
        Cd = empty_dev(m, words(n) + pad, fill=-1)
        product(bmm, sr)(to_dev(A, A.shape[1] + pad), to_dev(B), Cd, m, k, n,
                         options=bmm.Options(leaf=leaf, tile=1))
        got = from_dev(Cd)
        assert np.array_equal(got[:, :words(n)], want), (m, k, n)
        assert pad == 0 or (got[:, -1] == np.uint64(2**64 - 1)).all()  # past the row: untouched


@pytest.mark.parametrize("sname,sr", SEMIRINGS)
@pytest.mark.parametrize("fname,leaf", FORMATS)
def test_row_pitch_beyond_32_bit_offsets(bmm, sname, sr, fname, leaf):
    """Rows 2^20 words apart (8 MiB): row addresses are formed in 64 bits."""
    import torch
    m, k, n, ld = 130, 700, 70, 1 << 20
    A = bmmgen.fill_cpu(m, k, 5, bmmgen.TAG_A, bmmgen.Dist.inv_sqrt(k))
    B = bmmgen.fill_cpu(k, n, 5, bmmgen.TAG_B, bmmgen.Dist.inv_sqrt(k))
    announce("far rows", sname, fname)
    Ad = torch.zeros((m, ld), dtype=torch.int64, device="cuda")
    Ad[:, :words(k)] = to_dev(A)
    Cd = empty_dev(m, words(n), fill=-1)
    product(bmm, sr)(Ad, to_dev(B), Cd, m, k, n, options=bmm.Options(leaf=leaf, tile=1))
    assert np.array_equal(from_dev(Cd), oracle.mul(A, B, k, n, sr))


@pytest.mark.parametrize("fname,leaf,k", [("int8", 2, (1 << 24) - 1), ("fp4", 3, (1 << 24) - 1),
                                          ("int8", 2, (1 << 24) + 65)])
def test_longest_counts(bmm, fname, leaf, k):
    """All-ones rows: every count is k, the largest sum (2^7 k for int8); one row short of a
    bit, so that both parities occur.  int8 products of 2^24 and more take the other loop."""
    m, n = 3, 5
    A = np.full((m, words(k)), np.uint64(2**64 - 1))
    A[:, -1] &= np.uint64((1 << (k % 64)) - 1) if k % 64 else np.uint64(2**64 - 1)
    BT = np.repeat(A[:1], n, axis=0)
    A[1, 0] = A[1, 0] & ~np.uint64(1)
    A[2, :] = 0
    want = [k % 2, (k - 1) % 2, 0]
    for sr, bits in ((oracle.GF2, want), (oracle.BOOLEAN, [1, 1, 0])):
        announce("longest", fname, k, sr)
        Cd = empty_dev(m, 1, fill=-1)
        product(bmm, sr)(to_dev(A), to_dev(BT), Cd, m, k, n, b_transposed=True,
                         options=bmm.Options(leaf=leaf, tile=1))
        assert [int(x) for x in from_dev(Cd)[:, 0]] == [31 * b for b in bits]


# products of the small tiles: 64 x 64 with k split over four waves (up to 512 such tiles)
# and, from 513 of them, 128 x 128; k from one word to beyond the four waves' first stages
SMALL = [(64, 64, 64), (65, 2048, 65), (63, 2049, 200), (200, 1536, 63), (33, 5000, 300),
         (1, 1, 1), (1500, 577, 1500), (1537, 1024, 1473), (1600, 100, 1409)]


@pytest.mark.parametrize("sname,sr", SEMIRINGS)
@pytest.mark.parametrize("fname,leaf", FORMATS)
@pytest.mark.parametrize("tile", [2, 4])
def test_small_tiles(bmm, sname, sr, fname, leaf, tile):
    for i, (m, k, n) in enumerate(SMALL):
        p = bmmgen.Dist.half() if sr == oracle.GF2 else bmmgen.Dist.inv_sqrt(k)
        A = bmmgen.fill_cpu(m, k, 91 + i, bmmgen.TAG_A, p)
        B = bmmgen.fill_cpu(k, n, 91 + i, bmmgen.TAG_B, p)
        C0 = bmmgen.fill_cpu(m, n, 91 + i, 0xC0, bmmgen.Dist.half())
        ab = oracle.mul(A, B, k, n, sr)
        for acc in (False, True):
            announce("small", sname, fname, tile, (m, k, n), acc)
            Cd = to_dev(C0, words(n) + i % 2) if acc else empty_dev(m, words(n) + i % 2, fill=-1)
            product(bmm, sr)(to_dev(A, A.shape[1] + i % 2), to_dev(B), Cd, m, k, n,
                             options=bmm.Options(leaf=leaf, tile=tile), accumulate=acc)
            want = ab if not acc else (ab ^ C0 if sr == oracle.GF2 else ab | C0)
            assert np.array_equal(from_dev(Cd, words(n)), want), (m, k, n, acc)


# products that read B row-major in one launch (m k n up to 2^30, k up to 4096), and ones just
# past that; B's last rows short of a 64-row block, a stage and a wave's turn
ROWS = [(1, 1, 1), (64, 64, 64), (65, 63, 129), (130, 513, 70), (40, 2047, 200), (300, 4096, 257),
        (64, 4097, 64), (1024, 1024, 1024), (1025, 1024, 1024)]


@pytest.mark.parametrize("sname,sr", SEMIRINGS)
@pytest.mark.parametrize("fname,leaf", FORMATS)
@pytest.mark.parametrize("tile", [0, 2, 4])
def test_row_major_b_in_one_launch(bmm, sname, sr, fname, leaf, tile):
    for i, (m, k, n) in enumerate(ROWS):
        p = bmmgen.Dist.half() if sr == oracle.GF2 else bmmgen.Dist.inv_sqrt(k)
        A = bmmgen.fill_cpu(m, k, 111 + i, bmmgen.TAG_A, p)
        B = bmmgen.fill_cpu(k, n, 111 + i, bmmgen.TAG_B, p)
        C0 = bmmgen.fill_cpu(m, n, 111 + i, 0xC0, bmmgen.Dist.half())
        ab = oracle.mul(A, B, k, n, sr)
        for acc in (False, True):
            announce("rows", sname, fname, tile, (m, k, n), acc)
            Cd = to_dev(C0) if acc else empty_dev(m, words(n), fill=-1)
            product(bmm, sr)(to_dev(A, A.shape[1] + i % 2), to_dev(B, B.shape[1] + i % 3), Cd, m, k,
                             n, options=bmm.Options(leaf=leaf, tile=tile), accumulate=acc)
            want = ab if not acc else (ab ^ C0 if sr == oracle.GF2 else ab | C0)
            assert np.array_equal(from_dev(Cd, words(n)), want), (m, k, n, acc)


def test_transpose_edges(bmm):
    """Both tile sizes of the transpose (fewer than 256 tiles of 512 x 512 bits, or not), odd
    pitches, and edges within and past a 64-bit block; padding bits come out zero."""
    for i, (r, c) in enumerate([(1, 1), (64, 64), (65, 63), (257, 129), (511, 1025), (8200, 8129),
                                (16400, 4161)]):
        X = bmmgen.fill_cpu(r, c, 17 + i, bmmgen.TAG_A, bmmgen.Dist.half())
        for pad in (0, 1):
            announce("transpose", (r, c), pad)
            D = empty_dev(c, words(r) + pad, fill=-1)
            bmm.bmm_transpose(to_dev(X, X.shape[1] + pad), D, r, c)
            got = from_dev(D)
            bits = np.unpackbits(X.view(np.uint8), axis=1, bitorder="little")[:, :c]
            want = np.zeros((c, words(r) * 64), dtype=np.uint8)
            want[:, :r] = bits.T
            want = np.packbits(want, axis=1, bitorder="little").view(np.uint64)
            assert np.array_equal(got[:, :words(r)], want), (r, c, pad)
            assert pad == 0 or (got[:, -1] == np.uint64(2**64 - 1)).all()
