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


def kernels_of(call):
    """Names of the kernels that a call runs."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    return {e.name for e in p.events()}


# the option, or a record's choice where the option leaves it to that
@pytest.mark.parametrize("shift,record", [(1, None), (2, None), (-1, 1), (0, 1), (-1, None)])
@pytest.mark.parametrize("scheme", [0, 1])
@pytest.mark.parametrize("resident", [True, False])
def test_shifted_leaf_in_the_host_levels(bmm, tmp_path, shift, record, scheme, resident):
    import torch
    n, block = 8192, 4096  # leaves of 2048 bits
    if record is not None:
        table = tmp_path / "t.txt"
        table.write_text(f"depth {block} {block} {block} 1 0 {record}\n")
        bmm.bmm_autotune_load(str(table))
    A, B = operands(n, 61 + scheme)
    Ah, Bh = host(A), host(B)
    Ch = torch.full((n, words(n)), -1, dtype=torch.int64).pin_memory()
    announce("ooc shifted leaf", shift, record, scheme, resident)
    bmm.bmm_debug_fail_allocations(0 if resident else 1)  # the first one: A's place in HBM
    names = kernels_of(lambda: run(bmm, Ah, Bh, Ch, n, block, leaf=2, scheme=scheme, shift=shift))
    bmm.bmm_debug_fail_allocations(0)
    assert any("transpose_kernel" in x for x in names), names
    wanted = shift > 0 or (shift < 0 and bool(record))
    assert any("leaf_shift_kernel" in x for x in names) == wanted
    rows = bmmgen.stratified_rows(n, 128, 61)
    got = Ch.numpy().view(np.uint64)
    assert np.array_equal(got[rows], oracle.rows(A[rows], B, n, n, oracle.GF2))


@pytest.mark.parametrize("place", ["A", "B", "A and B", "rows of A"])
@pytest.mark.parametrize("resident", [True, False])
@pytest.mark.parametrize("n,block", [(1024, 256), (8192, 4096)])
def test_result_over_an_operand(bmm, place, resident, n, block):
    """The host levels read all of A and B before C goes down: a result written over them is
    still their product."""
    import torch
    A, B = operands(n, 71)
    if place == "A and B":
        B = A
    want = oracle.mul(A, B, n, n, oracle.GF2)
    tall = torch.zeros((n + n // 4, words(n)), dtype=torch.int64).pin_memory()
    tall[:n] = torch.from_numpy(A.view(np.int64))
    Ah = tall[:n]
    Bh = Ah if place == "A and B" else host(B)
    Ch = {"B": Bh, "rows of A": tall[n // 4:]}.get(place, Ah)
    announce("ooc over an operand", place, resident, n, block)
    bmm.bmm_debug_fail_allocations(0 if resident else 1)  # the first one: A's place in HBM
    got = run(bmm, Ah, Bh, Ch, n, block)
    bmm.bmm_debug_fail_allocations(0)
    assert np.array_equal(got, want)
