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


@pytest.mark.parametrize("rows,cols", [(8300, 8130), (300, 450)])  # large and small blocks
@pytest.mark.parametrize("start,src_pad,dst_pad", [(0, 1, 0), (1, 0, 1), (1, 1, 1), (0, 0, 0)])
def test_transpose_of_rows_at_8_bytes(bmm, rows, cols, start, src_pad, dst_pad):
    """Sources that start 8 bytes past a 16-byte line and pitches that keep rows there."""
    import torch
    X = bmmgen.fill_cpu(rows, cols, 11, bmmgen.TAG_A, bmmgen.Dist.half())
    ld = words(cols) + (words(cols) + src_pad) % 2  # odd where src_pad says so
    flat = torch.full((start + rows * ld,), -1, dtype=torch.int64, device="cuda")
    S = flat[start:].view(rows, ld)
    S[:, :words(cols)] = to_dev(X)
    D = empty_dev(cols, words(rows) + dst_pad, fill=-1)
    announce("transpose", rows, cols, start, src_pad, dst_pad)
    bmm.bmm_transpose(S, D, rows, cols)
    bits = np.unpackbits(X.view(np.uint8), axis=1, bitorder="little")[:, :cols]
    want = np.zeros((cols, words(rows) * 64), dtype=np.uint8)
    want[:, :rows] = bits.T
    got = from_dev(D)
    assert np.array_equal(got[:, :words(rows)],
                          np.packbits(want, axis=1, bitorder="little").view(np.uint64))
    assert dst_pad == 0 or (got[:, -1] == np.uint64(2**64 - 1)).all()


# a small product and products of few rows are one launch on a row-major B; the last ones,
# and a tile that is named or tuned, go through the scratch copy of B^T
@pytest.mark.parametrize("m,k,n,direct", [(256, 256, 256, True), (256, 64, 24576, True),
                                          (512, 600, 16384, True), (128, 64, 65536, False),
                                          (513, 64, 65536, False)])
@pytest.mark.parametrize("leaf", [2, 3])
@pytest.mark.parametrize("how", ["rule", "named", "tuned"])
def test_which_products_read_b_directly(bmm, m, k, n, direct, leaf, how):
    sr = oracle.GF2
    A, B = operands(m, k, n, sr, 23)
    bmm.bmm_finalize()  # no scratch, no tables
    if how == "tuned":
        bmm.bmm_autotune_set(sr, m, k, n, leaf, 5)
    o = bmm.Options(leaf=leaf, tile=5 if how == "named" else 0)
    C = empty_dev(m, words(n), fill=-1)
    Ad, Bd = to_dev(A), to_dev(B)
    announce("reads B directly", m, k, n, leaf, how)
    bmm.bmm_debug_fail_allocations(1)
    if direct and how == "rule":
        bmm.bmm_gf2(Ad, Bd, C, m, k, n, options=o)
    else:
        with pytest.raises(bmm.BmmError) as e:
            bmm.bmm_gf2(Ad, Bd, C, m, k, n, options=o)
        assert e.value.status == -4
        bmm.bmm_gf2(Ad, Bd, C, m, k, n, options=o)
    bmm.bmm_debug_fail_allocations(0)
    assert np.array_equal(from_dev(C), oracle.mul(A, B, k, n, sr))


@pytest.mark.parametrize("m,k,n", [(129, 513, 57345), (256, 1100, 32768), (400, 1024, 28672),
                                   (512, 2113, 16384)])
@pytest.mark.parametrize("leaf", [2, 3])
def test_few_rows_that_differ(bmm, m, k, n, leaf):
    """OR products of few rows in which every row of A has ones of its own, about two, so that
    a row in another's place shows."""
    sr = oracle.BOOLEAN
    rng = np.random.default_rng(m + k)
    A = np.zeros((m, words(k)), dtype=np.uint64)
    for j in rng.integers(0, k, (2, m)):
        A[np.arange(m), j // 64] |= np.uint64(1) << (j % 64).astype(np.uint64)
    B = bmmgen.fill_cpu(k, n, 29, bmmgen.TAG_B, bmmgen.Dist.half())
    want = oracle.mul(A, B, k, n, sr)
    assert len(np.unique(want, axis=0)) > m // 2
    C = empty_dev(m, words(n), fill=-1)
    announce("few rows that differ", m, k, n, leaf)
    bmm.bmm_boolean(to_dev(A), to_dev(B), C, m, k, n, options=bmm.Options(leaf=leaf))
    assert np.array_equal(from_dev(C), want)


@pytest.mark.parametrize("tall", [False, True])
def test_transpose_in_several_launches(bmm, tall):
    """One row (or column) of 2^32 + 700 bits: more 512 x 512 blocks than a launch takes."""
    import torch
    n = (1 << 32) + 700
    gen = torch.Generator(device="cuda").manual_seed(3)
    line = torch.randint(-(1 << 63), (1 << 63) - 1, (words(n),), dtype=torch.int64,
                         device="cuda", generator=gen)
    line[-1] &= (1 << (n % 64)) - 1
    shifts = torch.arange(64, device="cuda")
    step = 1 << 22  # words at a time
    announce("transpose in several launches", tall)
    if tall:
        src = torch.empty((n, 1), dtype=torch.int64, device="cuda")
        for i in range(0, words(n), step):
            part = ((line[i:i + step, None] >> shifts) & 1).flatten()
            src[64 * i:64 * i + part.numel(), 0] = part[:n - 64 * i]
        dst = torch.full((1, words(n)), -1, dtype=torch.int64, device="cuda")
        bmm.bmm_transpose(src, dst, n, 1)
        assert torch.equal(dst[0], line)
        return
    dst = torch.full((n, 1), -1, dtype=torch.int64, device="cuda")
    bmm.bmm_transpose(line[None, :], dst, 1, n)
    for i in range(0, words(n), step):
        part = ((line[i:i + step, None] >> shifts) & 1).flatten()[:n - 64 * i]
        assert torch.equal(dst[64 * i:64 * i + part.numel(), 0], part), i


# 528 and more tiles of 64 x 64, whole and ragged; one row, one column of them; k: a bit, words
# that fill steps of two and four of them and that do not, the last lengths before the next form
@pytest.mark.parametrize("m,n,ks", [(1472, 1473, (1, 64, 128, 193, 256, 257, 320, 321)),
                                    (300, 310, (1, 65, 128, 256)), (1, 1, (1, 200)),
                                    (33, 33000, (64, 700, 1024, 2047, 2048)),
                                    (33001, 64, (100, 513, 2040, 2050))])
@pytest.mark.parametrize("leaf", [2, 3])
@pytest.mark.parametrize("sr", [oracle.GF2, oracle.BOOLEAN])
def test_short_k_and_one_row_of_tiles(bmm, m, n, ks, leaf, sr):
    for k in ks:
        A, B = operands(m, k, n, sr, 31 + k)
        want = oracle.mul(A, B, k, n, sr)
        C0 = bmmgen.fill_cpu(m, n, 31 + k, 0xC0, bmmgen.Dist.half())
        BT = to_dev(np.zeros((n, words(k)), dtype=np.uint64))
        bmm.bmm_transpose(to_dev(B), BT, k, n)
        for pad, acc in ((0, False), (1, True), (2, False)):
            announce("short k", m, k, n, leaf, sr, pad, acc)
            C = empty_dev(m, words(n) + pad, fill=-1)
            if acc:
                C[:, :words(n)] = to_dev(C0)
            Bp = empty_dev(n, words(k) + pad, fill=-1)
            Bp[:, :words(k)] = BT
            product(bmm, sr)(to_dev(A, words(k) + pad), Bp, C, m, k, n, b_transposed=True,
                             accumulate=acc, options=bmm.Options(leaf=leaf))
            got = from_dev(C)
            ref = want if not acc else (want ^ C0 if sr == oracle.GF2 else want | C0)
            assert np.array_equal(got[:, :words(n)], ref), (k, pad, acc)
            assert (got[:, words(n):] == np.uint64(2**64 - 1)).all()


@pytest.mark.parametrize("leaf", [2, 3])
def test_result_of_2_to_the_36_bits(bmm, leaf):
    """Every named tile runs it, and the leaf tuner with them."""
    import torch
    m = n = 1 << 18
    k = 64
    A, B = operands(m, k, 64, oracle.GF2, 41)[0], operands(n, k, 64, oracle.GF2, 43)[0]  # B^T
    Ad, Bd = to_dev(A), to_dev(B)
    rows = bmmgen.stratified_rows(m, 64, 47)
    from oracle import brute
    want = oracle.rows(A[rows], brute.pack(brute.unpack(B, k).T.copy()), k, n, oracle.GF2)
    first = None
    for tile in (5, 2, 4):
        C = empty_dev(m, words(n), fill=-1)
        announce("2^36 bits", leaf, tile)
        bmm.bmm_gf2(Ad, Bd, C, m, k, n, b_transposed=True,
                    options=bmm.Options(leaf=leaf, tile=tile))
        if first is None:
            assert np.array_equal(from_dev(C[torch.from_numpy(np.asarray(rows, dtype=np.int64)).cuda()]), want)
            first = C
        else:
            assert torch.equal(C, first)
    if leaf == 3:
        announce("tuner, 2^36 bits")
        chosen, tile, secs = bmm.bmm_autotune_cubic(oracle.GF2, m, k, n)
        assert chosen in (1, 2, 3) and tile >= 1 and secs > 0
