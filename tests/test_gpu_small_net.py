"""The small-network kernel where its LDS ends: steps of more than 2048 key
slots and split lists of more than 1024 entries (D = 4, 5), more edges than next
crossings in LDS (65,000 vertices predicted, D = 2), no key slots (D = 1),
single neurons, layers of 32, 33 and 64 -- against the per-step kernels, bit for
bit, and the 256-thread batched kernel's counters."""
import numpy as np
import pytest

from paper_2306_07212_amd import workloads as wl

pytestmark = pytest.mark.gpu

SHAPES = [[1, 1, 1], [1, 64, 33, 1], [2, 1, 1, 1], [2, 32, 33, 1], [2, 64, 64, 64, 64, 64, 1], [3, 64, 1], [3, 33, 32, 1],
          [4, 27, 1], [5, 16, 1], [8, 3, 1]]


@pytest.mark.parametrize("widths", SHAPES)
def test_small_network_kernel_equals_the_per_step_kernels(monkeypatch, widths):
    from paper_2306_07212_amd import pcx
    net, box = wl.he_mlp(widths, [93, len(widths), widths[1]]), wl.cube(widths[0])
    m = pcx.MLP.from_net(net)
    monkeypatch.setenv("PCX_NO_TINY", "1")
    cx = pcx.extract(m, box.lo, box.hi)
    ref = (*cx.copy(), cx.steps())
    cx.close()
    for sched in (None, "0"):  # the small-network kernel; the 256-thread kernel, 32 lanes per split
        if sched is not None:
            monkeypatch.setenv("PCX_BATCH_SCHED", sched)
        bt = pcx.Batch([m, m], [(box.lo, box.hi)] * 2)
        st = bt.stats()
        print(f"[small] {widths} schedule {sched}: V={len(ref[0])} E={len(ref[2])} largest step "
              f"{ref[3][:, 2].max()} splits, fallbacks {st.fallbacks}", flush=True)
        for i in range(2):
            for a, b in zip((*bt.copy(i), bt.steps(i)), ref):
                assert a.shape == b.shape and np.array_equal(a, b), f"{widths} schedule {sched} network {i}"
        bt.close()
    m.close()


@pytest.mark.parametrize("widths", [[4, 5, 3, 1], [2, 17, 3, 1], [3, 16, 3, 1]])
def test_an_infinite_neuron_stays_out_of_the_others(monkeypatch, widths):
    """A first layer without crossings whose last neuron is infinite (an infinite bias): the second layer's are then
    infinite too, by the signs of their weights, and every vertex keeps them; the padding of the evaluation's inner
    dimension (K = 5, 17; 16 has none) must not turn them into NaN."""
    from paper_2306_07212_amd import pcx
    D, K, N = widths[0], widths[1], widths[2]
    W = [np.full((K, D), 0.01), np.ones((N, K)) * np.array([1.0, -1.0, 1.0])[:, None], np.ones((1, N))]
    b = [np.ones(K), np.zeros(N), np.zeros(1)]
    b[0][K - 1] = np.inf
    m, box = pcx.MLP(widths, W, b), wl.cube(D)
    for off in ("0", "1"):
        monkeypatch.setenv("PCX_NO_TINY", off)
        cx = pcx.extract(m, box.lo, box.hi)
        X, SG, Ed = cx.copy()
        cx.close()
        assert len(X) == 2**D and len(Ed) == D * 2 ** (D - 1)
        assert np.all(SG[:, -1] == 0b011001), f"{widths} PCX_NO_TINY={off}"  # +, -, + from bit 0 on
    m.close()


SMALL = [(4, [[4, n, 1] for n in range(3, 18, 2)] + [[4, 7, 8, 1], [4, 14, 2, 1], [4, 5, 5, 5, 1]]),
         (5, [[5, n, 1] for n in range(3, 11)] + [[5, 5, 5, 1], [5, 3, 3, 3, 1]]),
         (6, [[6, n, 1] for n in range(3, 8)] + [[6, 5, 1, 1], [6, 6, 1], [6, 3, 3, 1]]),
         (3, [[3, 1, 1], [3, 4, 1], [3, 9, 1], [3, 28, 1], [3, 14, 14, 1]])]


@pytest.mark.parametrize("D,shapes", SMALL, ids=[f"D{d}" for d, _ in SMALL])
@pytest.mark.parametrize("include_output", [False, True])
def test_small_networks_fit_their_room(monkeypatch, D, shapes, include_output):
    """Single networks of the sizes that go to the small-network kernel, from D = 4 on far above their predictions,
    fit its arena (no second extraction on the per-step path) and give the per-step kernels' complex."""
    from paper_2306_07212_amd import pcx
    box = wl.cube(D)
    for widths in shapes:
        for seed in range(4):
            m = pcx.MLP.from_net(wl.he_mlp(widths, [8, widths[1], seed]))
            bt = pcx.Batch([m], [(box.lo, box.hi)], include_output=include_output)
            assert bt.stats().fallbacks == 0, f"{widths} seed {seed}"
            with monkeypatch.context() as mp:
                mp.setenv("PCX_NO_TINY", "1")
                cx = pcx.extract(m, box.lo, box.hi, include_output=include_output)
            for a, b in zip((*bt.copy(0), bt.steps(0)), (*cx.copy(), cx.steps())):
                assert a.shape == b.shape and np.array_equal(a, b), f"{widths} seed {seed}"
            cx.close()
            bt.close()
            m.close()


@pytest.mark.parametrize("widths", [[4, 27, 1], [5, 16, 1], [6, 9, 1], [7, 4, 1], [8, 3, 1]])
def test_steps_past_the_lds_fit_the_arena(monkeypatch, widths):
    """Steps of more than 2048 key slots, and of more than 1024 splits (D = 4, 5), inside both kernels: nothing falls
    back, so what is compared with the per-step kernels is theirs."""
    from paper_2306_07212_amd import pcx
    m, box = pcx.MLP.from_net(wl.he_mlp(widths, [93, len(widths), widths[1]])), wl.cube(widths[0])
    monkeypatch.setenv("PCX_NO_TINY", "1")
    cx = pcx.extract(m, box.lo, box.hi)
    ref = (*cx.copy(), cx.steps())
    cx.close()
    largest = int(ref[3][:, 2].max())
    assert largest * 2 * (widths[0] - 1) > 2048 and (widths[0] > 5 or largest > 1024)
    for sched in (None, "0", "4"):
        if sched is not None:
            monkeypatch.setenv("PCX_BATCH_SCHED", sched)
        bt = pcx.Batch([m, m], [(box.lo, box.hi)] * 2)
        assert bt.stats().fallbacks == 0, f"{widths} schedule {sched}"
        for i in range(2):
            for a, b in zip((*bt.copy(i), bt.steps(i)), ref):
                assert a.shape == b.shape and np.array_equal(a, b), f"{widths} schedule {sched} network {i}"
        bt.close()
    m.close()


def test_a_network_that_outgrows_its_room_goes_per_step_from_then_on(oracle_lib):
    """Six layers that each fold the line four times: thousands of vertices where a He network of these sizes has
    dozens. The first extraction runs a second time on the per-step path; later ones go there at once, so that the
    repeats are replayed from the captured graph in the end. All are the same complex, the oracle's."""
    from paper_2306_07212_amd import pcx
    rng, L = np.random.default_rng(11), 6
    W = [np.ones((4, 1))] + [np.tile([4.0, -8.0, 8.0, -8.0], (4, 1)) * (1 + 1e-3 * rng.standard_normal((4, 4)))
                             for _ in range(L - 1)] + [np.ones((1, 4))]
    b = [-np.array([0.02, 0.25, 0.5, 0.75]) + 1e-3 * rng.standard_normal(4) for _ in range(L)] + [np.zeros(1)]
    net = wl.Net([1] + [4] * L + [1], W, b)
    lo, hi = np.zeros(1), np.ones(1)
    m = pcx.MLP.from_net(net)
    bt = pcx.Batch([m], [(lo, hi)])
    assert bt.stats().fallbacks == 1
    bt.close()
    got = []
    for _ in range(6):
        cx = pcx.extract(m, lo, hi)
        got.append((*cx.copy(), cx.steps()))
        graph = cx.info().from_graph
        cx.close()
    m.close()
    assert graph == 1
    for other in got[1:]:
        for x, y in zip(other, got[0]):
            assert x.shape == y.shape and np.array_equal(x, y)
    r = oracle_lib.extract(net, lo, hi)
    assert r.V == len(got[0][0]) and np.array_equal(got[0][3], r.steps)
