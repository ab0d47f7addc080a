"""GPU: contexts come and go. A context that is released, which Python may do at any moment, leaves a capture on
another stream intact and its host memory to later contexts; contexts alive together, on streams and
threads of their own, keep their sums apart."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPE = (20, 9, 7)


@pytest.fixture(scope="module")
def core():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_15781_amd import core as c

    c.lib()
    return c


def _sim(core, seed, stream=None):
    rng = np.random.default_rng(seed)
    solid = (rng.uniform(size=SHAPE[::-1]) < 0.3).astype(np.uint8)
    red = rng.uniform(0.1, 0.9, solid.shape)
    return core.Lbm(SHAPE, solid=solid, rho_r0=red, rho_p0=1 - red, precision="fp64", tau=0.8, sigma=0.02, beta=0.7,
                    xi=0.01, species=True, x_open=True, accel=[(1e-5, 0, 0)] * 2, stream=stream)


def test_release_during_a_capture(core):
    import torch

    stream = torch.cuda.Stream()
    sim, eager = _sim(core, 1, stream), _sim(core, 1)
    others = [_sim(core, k) for k in range(2, 5)]
    for o in others:
        o.step(2)
    start = sim.get_state()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        sim.advance(2)
        while others:
            others.pop().close()
        sim.advance(2)
    want = eager.step(12)
    for k in range(3):  # an even number of steps: every replay goes on from the state the last one left
        graph.replay()
        torch.cuda.synchronize()
        _sim(core, 9 + k).step(1)  # a new context takes a released one's memory between the replays
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(sim.populations(), eager.populations()))
    assert not torch.equal(start, sim.get_state())
    last = sim.state_sums()
    assert abs(last["mass_r"] + last["mass_p"] - (want[-1, 0] + want[-1, 1])) < 1e-9


def test_contexts_do_not_share_their_sums(core):
    """More contexts than are kept, twice; then four threads that make, step and release theirs."""
    alone = {k: _sim(core, k).step(3) for k in range(5)}
    for _ in range(2):
        sims = [_sim(core, k % 5) for k in range(20)]
        got = [s.step(1) for s in sims]
        for _ in range(2):
            got = [np.concatenate([g, s.step(1)]) for g, s in zip(got, sims)]
        for k, g in enumerate(got):
            assert np.array_equal(g, alone[k % 5]), k
        del sims
    wrong = []

    def work(k):
        import torch

        stream = torch.cuda.Stream()
        for _ in range(6):
            s = _sim(core, k, stream)
            if not np.array_equal(s.step(3), alone[k]):
                wrong.append(k)
            s.close()

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
