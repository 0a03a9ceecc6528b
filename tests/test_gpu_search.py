"""The forms of the search and of the compaction at the sizes where they
change: keys and units with as many moves as a lane, a wavefront or a
workgroup's list takes, lists that overflow, B with half of its states
single-arc (level search) and one more (chain search), few and many accepting
pairs, deep products, rows of a linear search, the limits of a small one, and
workspace caps.  Every array of C and the statistics against the oracle."""
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
@pytest.mark.parametrize("n", (7, 8, 9, 63, 64, 65, 130, 700))
def test_units_with_many_targets(order, n):
    """One arc of A against n arcs of B with its label, out of a state and
    back into it: targets taken by one lane (8 at most) or spread over all."""
    rng = np.random.default_rng(n)
    arcs = [(0, 1 + i, 1 + (i % 50 == 7), 1 + i % 3, float(rng.standard_normal()))
            for i in range(n)]
    arcs += [(1 + i, 0, 1 + (i % 40 == 3), 0, -0.5) for i in range(n)]
    arcs += [(1 + i, 1 + i, 1, 2, -1.5) for i in range(n)]  # two arcs a state: level search
    arcs += [(0, 1 + i, 0, 4, -1.0) for i in range(3)]
    B = synth.from_arcs(n + 1, arcs, start=[0], accept=[0, n])
    VA = 8200 // (n + 1) + 5  # more state pairs than a small search takes
    aarcs = [(t, (t + 1) % VA, 1, 1 + t % 2, 0.1 * (t % 3)) for t in range(VA)]
    aarcs += [(t, (t + 2) % VA, 2, 0 if t % 5 == 0 else 1, -0.2) for t in range(VA)]
    A = synth.from_arcs(VA, aarcs, start=[0, VA // 2], accept=[1, VA - 1])
    c = _composer(order)
    for X, Y in ((A, B), (B, A)):
        check_pair(c, X, Y, f"{n} targets {order}", ref=oracle.compose(X, Y, oracle.ORDER_FORWARD))
    c.close()


@pytest.mark.parametrize("order", ORDERS)
@pytest.mark.parametrize("chains", (0, 1))
def test_heavy_list_overflows(order, chains):
    """More heavy keys in a generation than the list's first size holds: the
    generations queued behind it must not read past the list."""
    from paper_2110_02848_amd import gpu
    rng = np.random.default_rng(17 + chains)
    A = synth.random_fst(rng, 170, 600, 9, 0.5, 0.1, start=range(30))
    arcs = [(s, (s + 1) % 50, 1 + s % 9, 1, 0.5) for s in range(50)]
    if not chains:
        arcs += [(s, (s + 7) % 50, 1 + s % 5, 2, 0.25) for s in range(50)]
    B = synth.from_arcs(50, arcs, start=range(50), accept=[9])
    ref = oracle.compose(A, B, oracle.ORDER_FORWARD)
    c = _composer(order)
    for cap in (1024, 256, 100, 1):  # whole pages of entries, and fewer
        c.set_option(gpu.FST_OPT_LIST_CAPACITY, cap)
        check_pair(c, A, B, f"heavy lists from {cap} {order} chains {chains}", ref=ref)
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


@pytest.mark.parametrize("order", ORDERS)
@pytest.mark.parametrize("p_accept", (0.02, 0.2, 0.25, 1.0))
@pytest.mark.parametrize("deep", (0, 1))
def test_backward_seeds(order, p_accept, deep):
    """Few accepting pairs to many (with more than half the words of the search
    bitmap, 5,120, the accessible keys are read instead: 300 states of which a
    quarter accept have 5,625), with f = 1 among them, forward searches of one
    generation and of many, B with several arcs a state and with one."""
    rng = np.random.default_rng(int(100 * p_accept) + deep)
    V, n_sym = 300, 3 if deep else 40
    A = synth.random_fst(rng, V, 4, n_sym, 0.1, 0.0, start=range(4))
    A["accept"][rng.permutation(V)[:int(p_accept * V)]] = 1
    for degree in (3, 1):
        B = synth.random_fst(rng, V, degree, n_sym, 0.1, 0.0, start=range(5))
        B["accept"][rng.permutation(V)[:int(p_accept * V)]] = 1
        c = _composer(order)
        check_pair(c, A, B, f"seeds {order} {p_accept} {deep} degree {degree}",
                   ref=oracle.compose(A, B, oracle.ORDER_FORWARD))
        c.close()


def _deep(rng, parts, VA):
    """A path of two-arc states through B with fans on the way: a part n > 0 is
    n such states, -n a state with n arcs (on several labels) to n states that
    meet again.  A: a few states that all have arcs of every label."""
    n_sym, arcs, s = 4, [], 0
    for n in parts:
        if isinstance(n, tuple):
            m, n = n
            for i in range(m):
                arcs.append((s, s + 1 + i, 1 + i % n_sym, 3, 0.1))
                for j in range(n):
                    t = s + 1 + m + i * n + j
                    arcs += [(s + 1 + i, t, 1 + j % n_sym, 1, 0.1), (t, s + 1 + m * (n + 1), 1, 2, 0.1),
                             (t, s + 1 + m * (n + 1), 2 + j % 3, 2, 0.3)]
            s += 1 + m * (n + 1)
        elif n > 0:
            for _ in range(n):
                arcs.append((s, s + 1, int(rng.integers(1, n_sym + 1)), 1, -0.1))
                arcs.append((s, s + 2, int(rng.integers(1, n_sym + 1)), 2, -0.2))
                s += 1
        else:
            n = -n
            for i in range(n):
                arcs.append((s, s + 3 + i, 1 + i % n_sym, 3, 0.1))
                arcs.append((s + 3 + i, s + 3 + n, 1 + i % 3, 0, -0.3))
                arcs.append((s + 3 + i, s + 3 + n, 0, 4, 0.2))
            arcs += [(s + 1, s + 3, 1, 1, 0.0), (s + 1, s + 4, 2, 1, 0.0),
                     (s + 2, s + 3, 3, 1, 0.0), (s + 2, s + 4, 2, 1, 0.0)]
            s += 3 + n
    B = synth.from_arcs(s + 3, arcs, start=[0], accept=[s, s + 1, s // 2])
    aarcs = [(a, (a + c) % VA, c, c, 0.1 * c) for a in range(VA) for c in range(1, n_sym + 1)]
    A = synth.from_arcs(VA, aarcs, start=[0], accept=range(VA))
    return A, B


@pytest.mark.parametrize("order", ORDERS)
@pytest.mark.parametrize("VA,parts", [
    (9, [1000]),                        # a few keys a wavefront all the way
    (16, [300, -200, 300]),             # a key of 200 units
    (3, [300, (20, 150), 400, (4, 200), 300]),  # hops that reach more than 64 keys
    (3, [1500, -254, 700, -255, 700, -256, 40, -257, 300, -600, 300]),  # heavy keys or just not
    (16, [300, -30, 20, -120, 60, -119, 100, -25, 25])])
def test_hops(order, VA, parts):
    """Deep products: wavefronts that go on with the keys they reached, until
    those are many, have many units or are heavy; and with work lists that
    overflow."""
    from paper_2110_02848_amd import gpu
    rng = np.random.default_rng(len(parts) + VA)
    A, B = _deep(rng, parts, VA)
    assert VA * B["num_states"] > 8192  # no small search
    ref = oracle.compose(A, B, oracle.ORDER_FORWARD)
    assert ref["num_states"] > 2000
    c = _composer(order)
    for k in range(2):
        check_pair(c, A, B, f"hops {VA} {parts} {order} call {k}", ref=ref)
    # generations past the 32nd reach many levels each
    assert 32 < c.stats()["fwd_levels"] < 32 + sum(p for p in parts if isinstance(p, int) and p > 0) // 4
    for cap in (64, 1):
        c.set_option(gpu.FST_OPT_LIST_CAPACITY, cap)
        check_pair(c, A, B, f"hops {VA} {parts} {order} lists from {cap}", ref=ref)
    c.close()


# ---- linear search: A's arcs lead from a state to the next, B mostly chains ----

def _frames(rng, T, C, p_gap=0.3, cuts=()):
    """Linear A of T frames: a random subset of the labels in each frame (some
    twice), no arc over the frames in cuts (utterances side by side)."""
    arcs = []
    for t in range(T):
        if t in cuts:
            continue
        for c in range(1, C + 1):
            for _ in range(1 if rng.random() < 0.9 else 2):
                if rng.random() >= p_gap:
                    arcs.append((t, t + 1, 1 + c % 3, c, float(rng.standard_normal())))
    start = [0] + [c + 1 for c in cuts] + ([T // 2] if T > 3 else [])
    return synth.from_arcs(T + 1, arcs, start=start, accept=[T, T // 3] + list(cuts))


def _words(rng, lens, C):
    """Words out of a root and back, as in a lexicon, some with epsilon inside."""
    arcs, s = [], 1
    for L in lens:
        arcs.append((0, s, 0, 1 + L % 5, 0.0))
        for _ in range(int(L)):
            arcs.append((s, s + 1, 0 if rng.random() < 0.1 else int(rng.integers(1, C + 1)), 0,
                         float(rng.standard_normal())))
            s += 1
        arcs.append((s, 0, 0, 0, -0.1))
        s += 1
    return synth.from_arcs(s, arcs, start=[0], accept=[0])


def _branches(rng, V, C):
    """Chains that split (a state that one arc leads to, with several) and
    meet again, dead ends, several start and accepting states."""
    arcs = []
    for s in range(V):
        x = rng.random()
        n = 1 if x < 0.7 else (0 if x < 0.75 else int(rng.integers(2, 5)))
        for i in range(n):
            d = s + 1 + i if rng.random() < 0.8 and s + 1 + i < V else int(rng.integers(0, V))
            arcs.append((s, d, 0 if rng.random() < 0.15 else int(rng.integers(1, C + 2)),
                         int(rng.integers(0, 4)), float(rng.standard_normal())))
    return synth.from_arcs(V, arcs, start=[0, V // 2], accept=[V - 1, V // 3, 0])


LINEAR = [("words", T) for T in (1, 2, 62, 63, 64, 65, 127, 128, 191, 4031, 4032, 4095)]
LINEAR += [("branches", T) for T in (1, 63, 64, 130, 4040)] + [("long words", 300)]


@pytest.mark.parametrize("kind,T", LINEAR)
def test_linear_search(kind, T):
    """Rows of one word to more than a wavefront's lanes, words (of the
    lexicon) shorter and longer than a chain record and than a thread's walk,
    frames that lack labels, utterances side by side: against the oracle, and
    with the walk cut short."""
    from paper_2110_02848_amd import gpu
    rng = np.random.default_rng(T)
    C = 5
    A = _frames(rng, T, C, p_gap=0.1 if T > 1000 else 0.3, cuts=(T // 2, T - 9) if T > 60 else ())
    if kind == "words":
        B = _words(rng, rng.integers(1, 7, size=12 if T > 1000 else 150), C)
    elif kind == "long words":
        B = _words(rng, [1, 2, 10, 11, 12, 13, 22, 23, 63, 64, 65, 66, 130, 200], 1)
        A = _frames(rng, T, 1, p_gap=0.0, cuts=(T - 9,))
    else:
        B = _branches(rng, 25 if T > 1000 else 90, C)
    ref = oracle.compose(A, B, oracle.ORDER_FORWARD)
    c = _composer("CONCURRENT")
    for depth in (64, 3, 1):
        c.set_option(gpu.FST_OPT_CHAIN_DEPTH, depth)
        check_pair(c, A, B, f"linear {kind} T={T} depth {depth}", ref=ref)
    c.set_option(gpu.FST_OPT_LIST_CAPACITY, 1)
    check_pair(c, A, B, f"linear {kind} T={T} lists from one entry", ref=ref)
    c.close()


def test_linear_search_without_room():
    """Workspace caps that leave no room for the rows, then none for lists of
    the first size: the keys are followed one by one, with shorter lists."""
    from paper_2110_02848_amd import gpu
    rng = np.random.default_rng(3)
    A, B = _frames(rng, 700, 4), _words(rng, rng.integers(1, 9, size=300), 4)
    ref = oracle.compose(A, B, oracle.ORDER_FORWARD)
    fits = []
    for cap in [1 << k for k in range(18, 28)]:
        c = _composer("CONCURRENT")
        c.set_option(gpu.FST_OPT_MAX_WORKSPACE, cap)
        try:
            check_pair(c, A, B, f"cap {cap}", ref=ref)
            fits.append(cap)
        except gpu.FstError as e:
            assert e.code == gpu.FST_ERR_NOMEM and not fits  # a larger cap never fails
        c.close()
    # the bitmaps (4 MB each), the views and short lists fit 32 MB
    assert fits and fits[0] <= 1 << 25


# ---- compaction by state ----

def _fans(rng, degrees, n_sym):
    """A graph whose state i has degrees[i] arcs (a few epsilon, labels with
    repeats), all to states drawn at random, every state accepting."""
    V = len(degrees)
    arcs = [(s, int(rng.integers(0, V)), int(rng.integers(0, n_sym + 1)) if rng.random() < 0.9
             else 0, int(rng.integers(1, n_sym + 1)) if rng.random() < 0.9 else 0,
             float(rng.standard_normal())) for s in range(V) for _ in range(int(degrees[s]))]
    return synth.from_arcs(V, arcs, start=range(V), accept=range(V))


@pytest.mark.parametrize("degrees", [(1,) * 64, (2,) * 65, (3,) * 63 + (40,), (33,) * 9,
                                     (31, 32, 33, 3, 4, 5, 7, 8, 9, 0, 1, 200), (6,) * 130])
@pytest.mark.parametrize("n_sym", (1, 3, 12))
def test_compaction_by_state(degrees, n_sym):
    """States with as many moves as a thread takes at a time (4), as make a
    state heavy (32) and as a wavefront's LDS holds (384), repeated labels on
    either side, the second call counting without waiting for the number of
    states, and a call without room for the list of keys."""
    from paper_2110_02848_amd import gpu
    rng = np.random.default_rng(len(degrees) + n_sym)
    A = _fans(rng, degrees, n_sym)
    B = _fans(rng, rng.integers(1, 5, size=6), n_sym)
    c = _composer("CONCURRENT")
    for X, Y in ((A, B), (B, A)):
        ref = oracle.compose(X, Y, oracle.ORDER_FORWARD)
        for k in range(2):
            check_pair(c, X, Y, f"by state {len(degrees)} {n_sym} call {k}", ref=ref)
    c.close()


def _walk_units(A, B, C):
    """Work units of C's states: epsilon arcs, and the other arcs of A, or of
    B where it has fewer (a quarter at most, or with different labels)."""
    def counts(g, lab):
        V = int(g["num_states"])
        eps = np.bincount(g["src"][g[lab] == 0], minlength=V)
        own = g["src"].astype(np.int64) * (int(g[lab].max()) + 1) + g[lab]
        v, n = np.unique(own[g[lab] > 0], return_counts=True)
        repeats = np.zeros(V, bool)
        repeats[v[n > 1] // (int(g[lab].max()) + 1)] = True
        return eps, np.bincount(g["src"], minlength=V) - eps, repeats
    (ea, na, _), (eb, nb, rep) = counts(A, "olabel"), counts(B, "ilabel")
    a, b = C["key_a"], C["key_b"]
    na, nb = na[a], nb[b]
    match = np.where((nb < na) & (~rep[b] | (na >= 4 * nb)), nb, na) * (nb > 0) * (na > 0)
    return np.where(C["key_f"] == 0, ea[a], 0) + eb[b] + match


@pytest.mark.parametrize("repeats_in_a", (0, 1))
@pytest.mark.parametrize("degree", (1, 2, 3, 4, 5, 8, 9, 31, 33))
def test_compaction_walks_the_side_with_fewer_arcs(repeats_in_a, degree):
    """States of B with a loop and arcs onward on the same label, against A's with
    many more arcs, their labels all different or not: the moves of a
    label in order, and no state with few units handed to a workgroup."""
    rng = np.random.default_rng(degree)
    V, n_sym = 120, 40 if not repeats_in_a else 17
    arcs = [(s, int(rng.integers(0, V)), 1 + i % 3, 1 + i % n_sym, float(rng.standard_normal()))
            for s in range(V) for i in range(40)]
    A = synth.from_arcs(V, arcs, start=range(V), accept=range(V))
    W, barcs = 90, []
    for s in range(W):
        labs = rng.integers(1, n_sym + 1, size=3)
        for i in range(degree):  # the first one a loop
            barcs.append((s, s if i == 0 else int(rng.integers(0, W)), int(labs[min(i // 2, 2)]),
                          int(rng.integers(0, 4)), float(rng.standard_normal())))
    B = synth.from_arcs(W, barcs, start=range(W), accept=range(W))
    c = _composer("CONCURRENT")
    for X, Y in ((A, B), (B, A)):
        ref = oracle.compose(X, Y, oracle.ORDER_FORWARD)
        for k in range(2):
            got, _ = check_pair(c, X, Y, f"loops {repeats_in_a} {degree} call {k}", ref=ref)
        assert c.stats()["heavy_states"] == int(np.sum(_walk_units(X, Y, got) > 32))
    c.close()


def test_count_launches():
    """What FST_OPT_TIMING reports of the count: a call that waits for the
    number of states, one that does not, one that has to count again, and
    empty results after each other."""
    import torch
    from paper_2110_02848_amd import gpu
    rng = np.random.default_rng(11)
    small = [synth.random_fst(rng, 150, 4, 5, 0.1, 0.3, start=range(9)) for _ in range(2)]
    large = [synth.random_fst(rng, 700, 5, 6, 0.1, 0.3, start=range(9)) for _ in range(2)]
    none = [synth.random_fst(rng, 200, 4, 5, 0.0, 0.0, start=range(9)) for _ in range(2)]
    none[0]["accept"][:] = none[1]["accept"][:] = 0
    c = _composer("CONCURRENT")
    c.set_option(gpu.FST_OPT_TIMING, 1)
    for pair, launches in ((small, 3), (small, 3), (large, 6), (large, 3), (none, 3), (none, 0),
                           (none, 0), (small, 3), (small, 3)):
        got, ref = check_pair(c, *pair, f"count of {pair[0]['num_states']}")
        torch.cuda.synchronize()
        ms, n = c.kernel_times()["count"]
        assert n == launches and (ms > 0) == (n > 0), (n, launches, ms)
    assert ref["num_states"] > 0
    c.close()


def test_compaction_without_room():
    """The least workspace cap that a call fits (to 64 KB): compaction by
    chunks; somewhat larger caps reach the list of keys."""
    from paper_2110_02848_amd import gpu
    rng = np.random.default_rng(9)
    A, B = (synth.random_fst(rng, 300, 4, 5, 0.1, 0.3, start=range(9)) for _ in range(2))
    ref = oracle.compose(A, B, oracle.ORDER_FORWARD)

    def fits(cap):
        c = _composer("CONCURRENT")
        c.set_option(gpu.FST_OPT_MAX_WORKSPACE, cap)
        try:
            for k in range(2):
                check_pair(c, A, B, f"cap {cap} call {k}", ref=ref)
            return True
        except gpu.FstError as e:
            assert e.code == gpu.FST_ERR_NOMEM
            return False
        finally:
            c.close()

    lo, hi = 1 << 16, 1 << 26
    assert fits(hi)
    while hi - lo > 1 << 16:
        mid = (lo + hi) // 2
        if fits(mid):
            hi = mid
        else:
            lo = mid
    for more in range(0, 12):
        assert fits(hi + more * (1 << 16)), more


# ---- workspace caps ----

def _least_cap(order, A, B, ref):
    """The least workspace cap (to 64 KB) that a fresh context composes in."""
    from paper_2110_02848_amd import gpu

    def fits(cap):
        c = _composer(order)
        c.set_option(gpu.FST_OPT_MAX_WORKSPACE, cap)
        try:
            check_pair(c, A, B, f"cap {cap}", ref=ref)
            return True
        except gpu.FstError as e:
            assert e.code == gpu.FST_ERR_NOMEM
            return False
        finally:
            c.close()

    lo, hi = 1 << 16, 1 << 27
    while hi - lo > 1 << 16:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if fits(mid) else (mid, hi)
    return hi


@pytest.mark.parametrize("order", ORDERS)
@pytest.mark.parametrize("kind", ("level", "linear", "chain"))
def test_workspace_of_earlier_calls(order, kind):
    """A call fits the cap that it fits in a fresh context also after larger
    calls, of every form of search, that left their buffers behind, and after
    calls that the cap refuses."""
    from paper_2110_02848_amd import gpu
    rng = np.random.default_rng(21)
    words = _words(rng, rng.integers(1, 9, size=120), 4)
    A, B = {"level": lambda: [synth.random_fst(rng, 200, 4, 5, 0.1, 0.3, start=range(9))
                              for _ in range(2)],
            "linear": lambda: (_frames(rng, 250, 4), words),
            "chain": lambda: (synth.random_fst(rng, 150, 5, 4, 0.1, 0.2, start=range(5)), words),
            }[kind]()
    ref = oracle.compose(A, B, oracle.ORDER_FORWARD)
    # (half as much again: how many keys a chain search hands on varies by run)
    cap = _least_cap(order, A, B, ref) * 3 // 2
    large = [[synth.random_fst(rng, 1500, 4, 6, 0.1, 0.3, start=range(9)) for _ in range(2)],
             [_frames(rng, 900, 4), _words(rng, rng.integers(1, 9, size=400), 4)]]
    refs = [oracle.compose(X, Y, oracle.ORDER_FORWARD) for X, Y in large]
    for (X, Y), r in zip(large, refs):
        c = _composer(order)
        check_pair(c, X, Y, f"large before {kind} {order}", ref=r)
        c.set_option(gpu.FST_OPT_MAX_WORKSPACE, cap)
        check_pair(c, A, B, f"{kind} {order} at {cap} after it", ref=ref)
        c.close()
        c = _composer(order)
        c.set_option(gpu.FST_OPT_MAX_WORKSPACE, cap)
        for k in range(2):
            with pytest.raises(gpu.FstError) as e:
                c.compose(gpu.to_device(X), gpu.to_device(Y))
            assert e.value.code == gpu.FST_ERR_NOMEM
            check_pair(c, A, B, f"{kind} {order} at {cap} after a refused call", ref=ref)
        c.close()


@pytest.mark.parametrize("order", ORDERS)
def test_lists_between_two_sizes(order):
    """A cap whose room for the work lists lies between a size that overflows
    and the next one that does not fit: every cap above the least one does."""
    from paper_2110_02848_amd import gpu
    rng = np.random.default_rng(5)
    A, B = (synth.random_fst(rng, 700, 4, 4, 0.1, 0.3, start=range(700)) for _ in range(2))
    ref = oracle.compose(A, B, oracle.ORDER_FORWARD)
    least = _least_cap(order, A, B, ref)
    for cap in [least + k * (least // 16) for k in range(16)]:
        c = _composer(order)
        c.set_option(gpu.FST_OPT_MAX_WORKSPACE, cap)
        check_pair(c, A, B, f"{order} lists in {cap}", ref=ref)
        c.close()


# ---- small search ----

def _search_launches(c):
    import torch
    torch.cuda.synchronize()
    return c.kernel_times()["search_forward"][1]


@pytest.mark.parametrize("VA,VB,starts,small", [
    (1, 1, 1, 1), (64, 128, 3, 1), (128, 64, 3, 1), (91, 90, 4, 1), (90, 91, 91, 0),
    (90, 91, 60, 0), (63, 65, 63, 1),
    # narrow operands whose search bitmaps (rows of 64 A states, columns of a
    # power of two of B states, 16 at least) still have at most 65,536 bits ...
    (2048, 1, 5, 1), (1, 512, 5, 1), (2000, 4, 3, 1), (33, 256, 4, 0),
    # ... and whose do not: another search
    (2049, 1, 5, 0), (8192, 1, 5, 0), (1, 513, 5, 0), (1, 8192, 5, 0), (3, 2730, 2, 0)])
def test_small_search(VA, VB, starts, small):
    """State pairs up to the limit of a small search (8192) and past it, levels
    of more keys than its lists hold (6144: every pair starts and accepts; then
    it is run again as a level search), narrow and wide operands, and which
    search it was (a small one is one launch)."""
    from paper_2110_02848_amd import gpu
    rng = np.random.default_rng(VA + VB)
    A = synth.random_fst(rng, VA, 3, 4, 0.2, 0.2 if starts < 60 else 1.0,
                         start=range(min(VA, starts)))
    B = synth.random_fst(rng, VB, 3, 4, 0.2, 0.2 if starts < 60 else 1.0,
                         start=range(min(VB, starts)))
    ref = oracle.compose(A, B, oracle.ORDER_FORWARD)
    c = _composer("CONCURRENT")
    c.set_option(gpu.FST_OPT_TIMING, 1)
    for k in range(2):
        check_pair(c, A, B, f"small {VA} {VB} {starts} call {k}", ref=ref)
        assert (_search_launches(c) == 1) == bool(small)
    c.close()


def _arcs_of(rng, V, arcs_a_state, n_sym, n_eps):
    """V states of that many arcs, n_eps of all with epsilon on both sides."""
    n = V * arcs_a_state
    il = rng.integers(1, n_sym + 1, size=n)
    il[rng.permutation(n)[:n_eps]] = 0
    arcs = [(i // arcs_a_state, int(rng.integers(0, V)), int(il[i]), int(il[i]),
             float(rng.standard_normal())) for i in range(n)]
    return synth.from_arcs(V, arcs, start=[0], accept=range(0, V, 3))


@pytest.mark.parametrize("VA,dA,eA,VB,dB,eB,small", [
    # units: epsilon arcs of A x VB, of B x VA (twice where A has some), and
    # the smaller of the other arcs x the other's states
    (64, 20, 0, 64, 20, 0, 1), (64, 20, 0, 64, 30, 0, 1),  # 81,920
    (64, 21, 0, 64, 21, 0, 0),                             # 86,016
    (64, 20, 1, 64, 20, 0, 1), (64, 20, 1, 64, 20, 1, 0),  # 81,920 and 81,984
    (20, 34, 0, 20, 34, 0, 1), (20, 35, 0, 20, 35, 0, 0),  # 13,600 and 14,000 of 13,696
    (1, 4120, 0, 1, 5000, 0, 1), (1, 4121, 0, 1, 4121, 0, 0), (1, 30000, 0, 1, 30000, 0, 0),
    (500, 4, 0, 1, 9000, 0, 1), (500, 4, 0, 1, 9000, 40, 0)])  # 2,000 and 20,000 more
def test_small_search_units(VA, dA, eA, VB, dB, eB, small):
    """Small searches end at a number of work units, over all pairs and per
    pair, whichever side they come from."""
    from paper_2110_02848_amd import gpu
    rng = np.random.default_rng(VA * dA + dB)
    n_sym = max(4, dA * dB // 4)
    A, B = _arcs_of(rng, VA, dA, n_sym, eA), _arcs_of(rng, VB, dB, n_sym, eB)
    ref = oracle.compose(A, B, oracle.ORDER_FORWARD)
    for validate in (1, 0):
        c = _composer("CONCURRENT")
        c.set_option(gpu.FST_OPT_TIMING, 1)
        c.set_option(gpu.FST_OPT_VALIDATE, validate)
        check_pair(c, A, B, f"units {VA} {dA} {eA} {VB} {dB} {eB}", ref=ref)
        assert (_search_launches(c) == 1) == bool(small)
        c.close()
