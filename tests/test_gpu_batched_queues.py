"""The persistent batched launch looks three items ahead and sets its own queue counters back:
plans of fewer items than queues, than workgroups and of several per workgroup, with k of
nothing, one and several stages, launched again and again and replayed from a graph."""
import numpy as np
import pytest

import bmmgen
import oracle
from oracle import brute
from gpu_util import announce, empty_dev, from_dev, to_dev, words

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bmm():
    import paper_1909_01554_amd as bmm
    return bmm


# (m, k, n) of the problems, repeated `times`; the semiring alternates
PLANS = {
    "one": ([(1, 1, 1)], 1),
    "nine": ([(300, 513, 200), (256, 0, 128), (257, 512, 129)], 3),
    "few_per_group": ([(520, 64, 300), (64, 1100, 1000), (256, 512, 128)], 60),
    "many_per_group": ([(1500, 200, 1500), (200, 4097, 70)], 30),
}


@pytest.mark.parametrize("name", sorted(PLANS))
@pytest.mark.parametrize("leaf,tile", [(2, 4), (3, 4), (3, 1), (2, 2), (3, 3)])
def test_queues_again_and_again(bmm, name, leaf, tile):
    import torch
    sizes, times = PLANS[name]
    data = []
    for j, (m, k, n) in enumerate(sizes):
        kk = max(k, 1)
        A = bmmgen.fill_cpu(m, kk, 70 + j, bmmgen.TAG_A, bmmgen.Dist.half())
        BT = bmmgen.fill_cpu(n, kk, 70 + j, bmmgen.TAG_B, bmmgen.Dist.half())
        B = brute.pack(brute.unpack(BT, kk).T.copy())
        want = [oracle.mul(A, B, k, n, sr) if k else np.zeros((m, words(n)), np.uint64)
                for sr in (oracle.GF2, oracle.BOOLEAN)]
        data.append((to_dev(A), to_dev(BT), want))
    probs, wants = [], []
    for i in range(times):
        for (m, k, n), (A, BT, want) in zip(sizes, data):
            sr = (i + len(probs)) % 2
            probs.append(dict(semiring=sr, m=m, k=k, n=n, A=A, B=BT,
                              C=empty_dev(m, words(n), fill=-1), b_transposed=True))
            wants.append(want[(oracle.GF2, oracle.BOOLEAN).index(sr)])
    announce("batched queues", name, leaf, tile)
    plan = bmm.BatchedPlan(probs, options=bmm.Options(leaf=leaf, tile=tile))

    def check():
        torch.cuda.synchronize()
        for p, want in zip(probs, wants):
            assert np.array_equal(from_dev(p["C"], words(p["n"])), want)
            p["C"].fill_(-1)
        torch.cuda.synchronize()

    for _ in range(2):
        plan.launch()
        check()
    for _ in range(3):
        plan.launch()
    check()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.launch()
        plan.launch()
    for _ in range(3):
        graph.replay()
        check()
        plan.launch()
        check()
    plan.destroy()
