"""The out-of-core product under tuned depth records, options and aliased host operands,
bit-exact against the oracle."""
import numpy as np
import pytest

import bmmgen
import oracle
from gpu_util import announce, words

pytestmark = pytest.mark.gpu


@pytest.fixture
def bmm():
    import paper_1909_01554_amd as bmm
    bmm.bmm_finalize()
    yield bmm
    bmm.bmm_debug_fail_allocations(0)
    bmm.bmm_finalize()


def operands(n, seed):
    return [bmmgen.fill_cpu(n, n, seed, tag, bmmgen.Dist.half())
            for tag in (bmmgen.TAG_A, bmmgen.TAG_B)]


def host(x):
    import torch
    return torch.from_numpy(x.view(np.int64).copy()).pin_memory()


def run(bmm, Ah, Bh, Ch, n, block, **kw):
    bmm.bmm_ooc(oracle.GF2, Ah, Bh, Ch, n, n, n, block=block, options=bmm.Options(**kw))
    return Ch.numpy().view(np.uint64)


@pytest.mark.parametrize("block_order", [False, True])
@pytest.mark.parametrize("depth,ds", [(2, 2), (2, 1), (2, 0), (1, 1)])
def test_depth_record_of_the_block(bmm, tmp_path, depth, ds, block_order):
    """A record's split is what runs, in the workspace that was planned for it."""
    import torch
    n, block = 1024, 512
    table = tmp_path / "t.txt"
    table.write_text(f"depth {block} {block} {block} {depth} {ds} 0\n")
    bmm.bmm_autotune_load(str(table))
    A, B = operands(n, 51 + depth + ds)
    Ch = torch.full((n, words(n)), -1, dtype=torch.int64).pin_memory()
    announce("ooc depth record", depth, ds, block_order)
    got = run(bmm, host(A), host(B), Ch, n, block,
              flags=bmm.FLAG_OOC_BLOCK_ORDER if block_order else 0)
    assert np.array_equal(got, oracle.mul(A, B, n, n, oracle.GF2))
