"""The VALU leaf with B passed transposed takes no scratch: neither the default rule nor a
table entry picks the form that reads B row-major (it would turn B back into the buffer that
calls on other streams share); only a caller that names that tile gets it."""
import os
import subprocess
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TABLE = os.path.join(ROOT, "paper_1909_01554_amd", "tune_gfx950.txt")
BIG = [(16384, 16384, 16384), (12700, 300, 12700), (1 << 18, 1 << 18, 1 << 18)]


@pytest.fixture
def bmm():
    import paper_1909_01554_amd as bmm
    bmm.bmm_finalize()
    yield bmm
    bmm.bmm_debug_fail_allocations(0)
    bmm.bmm_finalize()


@pytest.mark.parametrize("table", [False, True])
@pytest.mark.parametrize("m,k,n", BIG)
def test_choice_follows_the_form_of_b(bmm, m, k, n, table):
    if table:
        bmm.bmm_autotune_load(TABLE)
    for sr in (bmm.GF2, bmm.BOOLEAN):
        given_t = bmm.Options(leaf=bmm.LEAF_VALU, flags=bmm.FLAG_B_TRANSPOSED)
        assert bmm.bmm_leaf_choice(sr, m, k, n, options=given_t) == (bmm.LEAF_VALU, 1)
        given = bmm.Options(leaf=bmm.LEAF_VALU)
        assert bmm.bmm_leaf_choice(sr, m, k, n, options=given) == (bmm.LEAF_VALU, 2)


def test_tuned_entry_and_named_tile(bmm):
    """An entry's tile 2 was timed on a row-major B and serves those; a named tile is kept."""
    m, k, n = 640, 512, 768
    bmm.bmm_autotune_set(bmm.GF2, m, k, n, bmm.LEAF_VALU, 2)
    assert bmm.bmm_leaf_choice(bmm.GF2, m, k, n) == (bmm.LEAF_VALU, 2)
    t = bmm.Options(flags=bmm.FLAG_B_TRANSPOSED)
    assert bmm.bmm_leaf_choice(bmm.GF2, m, k, n, options=t) == (bmm.LEAF_VALU, 1)
    t.leaf, t.tile = bmm.LEAF_VALU, 2
    assert bmm.bmm_leaf_choice(bmm.GF2, m, k, n, options=t) == (bmm.LEAF_VALU, 2)


NO_DEVICE = """
import ctypes, sys
import torch
if torch.cuda.device_count():
    sys.exit(77)
import paper_1909_01554_amd as bmm
bmm.bmm_autotune_load(sys.argv[1])
n = 1 << 18
o = bmm.Options(leaf=bmm.LEAF_VALU, flags=int(sys.argv[2]))
vp = ctypes.c_void_p
size = n * n // 8
rc = bmm._c_noalloc(1, vp(size), n // 64, vp(3 * size), n // 64, vp(5 * size), n // 64, n, n, n,
                    ctypes.byref(o), None)
print(rc, bmm._c_last_error().decode())
"""


@pytest.mark.parametrize("given_transposed,entry", [(True, None), (True, 2), (False, None)])
def test_noalloc_at_a_table_entry(bmm, tmp_path, given_transposed, entry):
    """The entry point without allocations at 2^18, with the shipped table and with an entry
    that names tile 2 (no device in the child: the addresses are never read): B^T reaches the
    leaf launch, B is too large to stage."""
    table = TABLE
    if entry:
        table = tmp_path / "t.txt"
        table.write_text(f"leaf 1 {1 << 18} {1 << 18} {1 << 18} 1 1 {entry} 0 0\n")
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1", CUDA_VISIBLE_DEVICES="-1")
    flags = bmm.FLAG_B_TRANSPOSED if given_transposed else 0
    r = subprocess.run([sys.executable, "-c", NO_DEVICE, str(table), str(flags)], cwd=ROOT,
                       env=env, capture_output=True, text=True, timeout=300)
    if r.returncode == 77:
        pytest.skip("devices cannot be hidden")
    assert r.returncode == 0, r.stderr[-2000:]
    status, message = r.stdout.strip().splitlines()[-1].split(" ", 1)
    if given_transposed:
        assert int(status) == -5 and message.startswith("leaf launch"), r.stdout
    else:
        assert int(status) == -2 and "staging" in message, r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("sr", [0, 1])
def test_no_scratch_with_b_transposed(bmm, sr):
    import bmmgen
    import oracle
    from gpu_util import announce, empty_dev, from_dev, to_dev, words
    m, k, n = 12700, 145, 12673
    dist = bmmgen.Dist.half() if sr == oracle.GF2 else bmmgen.Dist.inv_sqrt(k)
    A = bmmgen.fill_cpu(m, k, 19, bmmgen.TAG_A, dist)
    B = bmmgen.fill_cpu(k, n, 19, bmmgen.TAG_B, dist)
    want = oracle.mul(A, B, k, n, sr)
    BT = to_dev(np.zeros((n, words(k)), dtype=np.uint64))
    bmm.bmm_transpose(to_dev(B), BT, k, n)
    fn = bmm.bmm_gf2 if sr == oracle.GF2 else bmm.bmm_boolean
    announce("VALU leaf, B transposed, no scratch", sr)
    C = empty_dev(m, words(n), fill=-1)
    Ad = to_dev(A)
    bmm.bmm_debug_fail_allocations(1)  # any scratch would have to be allocated
    fn(Ad, BT, C, m, k, n, options=bmm.Options(leaf=1), b_transposed=True)
    bmm.bmm_debug_fail_allocations(0)
    assert np.array_equal(from_dev(C), want)
    # the named tile still turns B back, and gives the same product
    C2 = empty_dev(m, words(n), fill=-1)
    fn(Ad, BT, C2, m, k, n, options=bmm.Options(leaf=1, tile=2), b_transposed=True)
    assert np.array_equal(from_dev(C2), want)
