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
