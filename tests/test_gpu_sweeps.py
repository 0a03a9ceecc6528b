"""Relaxation sweeps at the sizes where a wavefront's share changes: 64
consecutive states whose arcs just fit its LDS (512) or do not, a last
wavefront that is full, one state short or one state long, states without
arcs, and graphs most of whose values do not change from sweep to sweep."""
import numpy as np
import pytest

from paper_2110_02848_amd import synth

from test_gpu_score_cyclic import _check, _run, comp, settled_sweep  # noqa: F401 (a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", (1, 63, 64, 65, 128, 129))
@pytest.mark.parametrize("degree", (1, 8, 9))
def test_edges_of_a_wavefront(comp, V, degree):  # noqa: F811
    G = synth.random_cyclic(100 + V, V, degree=degree, mass=0.5)
    _check(comp, G, f"V={V} degree {degree}")
    if degree == 8 and V >= 64:  # one arc more in the first 64 states
        arcs = list(zip(G["src"], G["dst"], G["ilabel"], G["olabel"], G["weight"]))
        arcs.append((5, V - 1, 1, 1, np.float32(-6.0)))
        H = synth.from_arcs(V, arcs, start=np.nonzero(G["start"])[0],
                            accept=np.nonzero(G["accept"])[0])
        _check(comp, H, f"V={V} 513 arcs")


@pytest.mark.parametrize("gap", (1, 3))
def test_values_that_settle_at_different_sweeps(comp, gap):  # noqa: F811
    """A long chain in front of a small cyclic part, and states without
    arcs between: after the first sweeps a few states at a time change.  The
    chain's values equal fst_score's bit for bit (it has no cycle)."""
    import torch
    from paper_2110_02848_amd import gpu
    n = 700
    arcs = [(gap * i, gap * (i + 1), 1, 1, -0.01 * (i % 7)) for i in range(n)]
    arcs += [(gap * i, gap * (i + 2), 1, 1, -0.5) for i in range(0, n - 2, 5)]
    V = gap * n + 3
    chain = synth.from_arcs(V, arcs, start=[0], accept=[gap * n])
    got = _run(comp, chain)
    ref = comp.score(gpu.to_device(chain))
    torch.cuda.synchronize()
    for k in ("alpha", "beta"):
        assert np.array_equal(got[k].view(np.int64), ref[k].cpu().numpy().view(np.int64)), k
    # (the paths with the most arcs add less than a unit in the last place)
    assert got["sweeps"] == settled_sweep(chain) < n + 2
    loop = arcs + [(gap * n, gap * n + 1, 1, 1, -1.0), (gap * n + 1, gap * n, 1, 1, -0.7)]
    _check(comp, synth.from_arcs(V, loop, start=[0], accept=[gap * n]), f"chain and cycle {gap}")


@pytest.mark.parametrize("V", (1, 2, 8, 20, 64, 65, 100, 700))
@pytest.mark.parametrize("dirs", ((True, True), (True, False), (False, True)))
def test_the_sweep_that_settled(comp, V, dirs):  # noqa: F811
    """A path of V states ends in a state that nobody pulls from (the start
    state, backward): sweep V gives it its value, sweep V + 1 raises none and
    is the one that settled, wherever a batch of sweeps ends."""
    G = synth.from_arcs(V, [(i, i + 1, 1, 1, -0.01 * (i % 7)) for i in range(V - 1)], start=[0],
                        accept=[V - 1])
    assert settled_sweep(G) == V + 1
    for tol in (0.0, 0.5):
        got = _run(comp, G, alpha=dirs[0], beta=dirs[1], tol=tol)
        assert got["sweeps"] == V + 1, (got["sweeps"], V, tol)
    # no sweep more is needed, and one less is not enough
    assert _run(comp, G, alpha=dirs[0], beta=dirs[1], max_sweeps=V + 1)["sweeps"] == V + 1
    from paper_2110_02848_amd import gpu
    with pytest.raises(gpu.FstError) as e:
        _run(comp, G, alpha=dirs[0], beta=dirs[1], max_sweeps=V)
    assert e.value.code == gpu.FST_ERR_NOT_CONVERGED


@pytest.mark.parametrize("degree", (1, 3, 8, 9, 20))
def test_without_room_for_ranks(comp, degree):  # noqa: F811
    """The least workspace cap that fits: the arcs' ranks share the values'
    room (8 arcs a state and fewer) or are done without; the same bits."""
    from paper_2110_02848_amd import gpu
    V = 3000
    G = synth.random_cyclic(degree, V, degree=degree, mass=0.5)
    want = _run(comp, G)

    def at(cap):
        c = gpu.Composer(0)
        c.set_option(gpu.FST_OPT_MAX_WORKSPACE, cap)
        try:
            return _run(c, G)
        except gpu.FstError as e:
            assert e.code == gpu.FST_ERR_NOMEM
            return None
        finally:
            c.close()

    lo, hi = 1 << 12, 1 << 24
    while hi - lo > 1 << 12:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if at(mid) else (mid, hi)
    # in-arcs 8 bytes an arc and 4 a state, values 32, bits 1/2, notes 41 KB and
    # at most 12 KB of scan and rounding
    assert hi < 8 * degree * V + 36.5 * V + (56 << 10), hi
    for cap in (hi, hi + degree * V * 2, hi + degree * V * 4 + 4096):
        got = at(cap)
        assert got["sweeps"] == want["sweeps"]
        for k in ("alpha", "beta"):
            assert np.array_equal(got[k].view(np.int64), want[k].view(np.int64)), (k, cap)
