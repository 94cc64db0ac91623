"""The largest results a named matrix-core tile is launched for.  Only the host's checks run:
the calls are made in a child without a device, on addresses that are never read."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import ctypes, sys
import torch
if torch.cuda.device_count():
    sys.exit(77)
import paper_1909_01554_amd as bmm
m, k, n = (int(x) for x in sys.argv[1:4])
pitch = int(sys.argv[6])
o = bmm.Options(leaf=int(sys.argv[4]), tile=int(sys.argv[5]), flags=bmm.FLAG_B_TRANSPOSED)
vp, base = ctypes.c_void_p, 1 << 56
rc = bmm._c_gf2(vp(base), pitch, vp(2 * base), pitch, vp(3 * base), n // 64, m, k, n,
                ctypes.byref(o), None)
print(rc, bmm._c_last_error().decode())
"""


def status(m, k, n, leaf, tile, pitch=0):
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1", CUDA_VISIBLE_DEVICES="-1")
    args = [str(x) for x in (m, k, n, leaf, tile, pitch or k // 64)]
    r = subprocess.run([sys.executable, "-c", CHILD] + args, cwd=ROOT, env=env,
                       capture_output=True, text=True, timeout=300)
    if r.returncode == 77:
        pytest.skip("devices cannot be hidden")
    assert r.returncode == 0, r.stderr[-2000:]
    rc, message = r.stdout.strip().splitlines()[-1].split(" ", 1)
    assert message.startswith("leaf launch"), r.stdout
    return int(rc)


# 2^24 tiles of 64 x 64 (2^32 work-items), and one more row of them
@pytest.mark.parametrize("m,n", [(1 << 18, 1 << 18), ((1 << 18) + 1, 1 << 18)])
@pytest.mark.parametrize("leaf", [2, 3])
@pytest.mark.parametrize("tile", [2, 4])
def test_small_tiles_reach_their_launch(m, n, leaf, tile):
    assert status(m, 64, n, leaf, tile) == -5  # no device: the launch itself fails


# 2^24 workgroups of 2 x 2 wave tiles of the named size
@pytest.mark.parametrize("m,n,tile", [(1 << 20, 1 << 18, 2), (1 << 19, 1 << 18, 4),
                                      ((1 << 31) - 64, 64, 2), (64, 1 << 30, 4)])
@pytest.mark.parametrize("pitch", [32, 1 << 20])
@pytest.mark.parametrize("leaf", [2, 3])
def test_past_the_named_tiles_is_refused(m, n, tile, pitch, leaf):
    assert status(m, 2048, n, leaf, tile, pitch) == -2


def test_past_the_panel_tiles_is_refused():
    assert status(1 << 20, 64, 1 << 19, 3, 4) == -2


# one column or row of tiles, twice as many as the register-fed form can launch
@pytest.mark.parametrize("leaf", [2, 3])
@pytest.mark.parametrize("m,k,n", [((1 << 31) - 64, 64, 64), ((1 << 31) - 64, 2048, 64),
                                   (64, 64, (1 << 31) - 64)])
def test_default_tile_of_a_single_column_can_be_launched(m, k, n, leaf):
    assert status(m, k, n, leaf, 0) == -5


def test_default_tile_of_a_large_batch_can_be_launched():
    """7^7 leaves of 600 x 600: 25 tiles of 128 x 128 each would be too many work-items, 15 of
    128 x 256 are not."""
    import paper_1909_01554_amd as bmm
    for leaf in (bmm.LEAF_MFMA_I8, bmm.LEAF_MFMA_F4):
        o = bmm.Options(leaf=leaf)
        assert bmm.bmm_leaf_choice(bmm.GF2, 600, 512, 600, batch=7 ** 4, options=o)[1] == 2
        assert bmm.bmm_leaf_choice(bmm.GF2, 600, 512, 600, batch=7 ** 7, options=o)[1] != 2


TRANSPOSE = """
import ctypes, sys
import torch
if torch.cuda.device_count():
    sys.exit(77)
import paper_1909_01554_amd as bmm
rows, cols = int(sys.argv[1]), int(sys.argv[2])
vp, base = ctypes.c_void_p, 1 << 44
print(bmm._c_transpose(vp(base), (cols + 63) // 64, vp(2 * base), (rows + 63) // 64, rows, cols,
                       None))
"""


# 512 x 512 bits per workgroup of 512 threads: 2^23 of them in several launches, 2^24 refused
@pytest.mark.parametrize("rows,cols,want", [(64, 1 << 32, -5), (1 << 32, 64, -5),
                                            (1, (1 << 33) - 513, -5), (64, 1 << 33, -2)])
def test_transposes_past_one_launch(rows, cols, want):
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1", CUDA_VISIBLE_DEVICES="-1")
    r = subprocess.run([sys.executable, "-c", TRANSPOSE, str(rows), str(cols)], cwd=ROOT, env=env,
                       capture_output=True, text=True, timeout=300)
    if r.returncode == 77:
        pytest.skip("devices cannot be hidden")
    assert r.returncode == 0, r.stderr[-2000:]
    assert int(r.stdout.strip().splitlines()[-1]) == want
