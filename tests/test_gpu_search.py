"""The two kinds of search, level and chain, at the sizes where they change:
keys with as many moves as a wavefront takes, a workgroup's list holds and a
generation hands on; B with half of its states single-arc (level search) and
one more (chain search); frontiers of a few keys and of many.  Every array
of C and the statistics against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2110_02848_amd import synth

from test_gpu_parity import check_pair

pytestmark = pytest.mark.gpu

ORDERS = ("FORWARD_FIRST", "COACCESSIBLE_FIRST", "CONCURRENT")


def _composer(order):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2110_02848_amd import gpu
    c = gpu.Composer(0)
    c.set_option(gpu.FST_OPT_ORDER, getattr(gpu, "FST_ORDER_" + order))
    c.set_option(gpu.FST_OPT_COUNT_MOVES, 1)
    return c


def _hubs(rng, fans):
    """A with a hub of each fan-out (epsilon and matching arcs) whose arcs
    lead to one middle layer and back to the hubs; B with two or more arcs a
    state."""
    arcs, mid = [], len(fans)
    for h, n in enumerate(fans):
        for i in range(n):
            arcs.append((h, mid + int(rng.integers(0, 40)), 1 + i % 5,
                         0 if i % 3 else 1 + i % 4, float(rng.standard_normal())))
    for m in range(40):
        arcs.append((mid + m, int(rng.integers(0, len(fans))), 2, 1 + m % 4, 0.5))
        arcs.append((mid + m, mid + int(rng.integers(0, 40)), 3, 0, -0.25))
    A = synth.from_arcs(mid + 40, arcs, start=range(len(fans)), accept=range(mid, mid + 7))
    B = synth.tiny_random(rng, 9, 6, 4, 0.3)
    return A, B


@pytest.mark.parametrize("order", ORDERS)
@pytest.mark.parametrize("fans", [(1, 2, 63), (64, 65, 66), (255, 256, 257), (300, 1024, 5000)])
def test_keys_with_many_moves(order, fans):
    A, B = _hubs(np.random.default_rng(fans[0]), fans)
    c = _composer(order)
    check_pair(c, A, B, f"hubs {fans} {order}", ref=oracle.compose(A, B, oracle.ORDER_FORWARD))
    # the same pair the other way round: the hubs on B's side, no epsilon input
    check_pair(c, B, A, f"hubs in B {fans} {order}", ref=oracle.compose(B, A, oracle.ORDER_FORWARD))
    c.close()


@pytest.mark.parametrize("order", ORDERS)
@pytest.mark.parametrize("more", (0, 1))
def test_single_arc_states_of_b(order, more):
    """n states of B with one arc among 2 n (level search) or 2 n - 1."""
    rng = np.random.default_rng(5 + more)
    n, V = 40, 80 - more
    arcs = []
    for s in range(V):
        for _ in range(1 if s < n else int(rng.integers(2, 5))):
            arcs.append((s, int(rng.integers(0, V)), int(rng.integers(0, 6)),
                         int(rng.integers(0, 6)), float(rng.standard_normal())))
    B = synth.from_arcs(V, arcs, start=[0, 7], accept=[3, V - 1])
    A = synth.random_fst(rng, 70, 4, 5, 0.1, 0.1, start=(0, 1, 2))
    c = _composer(order)
    check_pair(c, A, B, f"single arcs {more} {order}", ref=oracle.compose(A, B, oracle.ORDER_FORWARD))
    c.close()
