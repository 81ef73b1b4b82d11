"""Single networks with layers wider than 64 that go to one workgroup (on the
line; in the plane behind a first layer of at most 10 neurons) and their
neighbours that do not, against the per-step kernels, bit for bit."""
import numpy as np
import pytest

from paper_2306_07212_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("widths", [[1, 65, 1], [1, 204, 256, 1], [2, 10, 65, 1], [2, 10, 110, 1], [2, 11, 65, 1],
                                    [2, 10, 120, 1], [2, 2, 3, 100, 1]])
@pytest.mark.parametrize("include_output", [False, True])
def test_wide_layers_of_a_single_network(monkeypatch, widths, include_output):
    from paper_2306_07212_amd import pcx
    m, box = pcx.MLP.from_net(wl.he_mlp(widths, [97, sum(widths)])), wl.cube(widths[0])
    got = []
    for off in ("0", "1"):
        monkeypatch.setenv("PCX_NO_TINY", off)
        cx = pcx.extract(m, box.lo, box.hi, include_output=include_output)
        got.append((*cx.copy(), cx.steps()))
        cx.close()
    m.close()
    print(f"[wide] {widths}: V={len(got[0][0])} E={len(got[0][2])}", flush=True)
    for a, b in zip(*got):
        assert a.shape == b.shape and np.array_equal(a, b)


@pytest.mark.parametrize("widths,one_workgroup", [
    ([1, 65, 1], True), ([1, 204, 256, 1], True), ([2, 4, 100, 1], True), ([2, 10, 65, 1], True), ([2, 30, 2, 90, 1], True),
    ([2, 8, 8, 8, 100, 1], True), ([2, 10, 100, 1], False), ([2, 16, 65, 1], False), ([2, 65, 1], False),
    ([2, 100, 30, 1], False), ([3, 4, 65, 1], False)])
def test_route_of_wide_layers(widths, one_workgroup):
    """Only the per-step path is captured, so repeats tell the two apart; what goes to one workgroup fits it (no
    second extraction), and all repeats are the same complex."""
    from paper_2306_07212_amd import pcx
    m, box = pcx.MLP.from_net(wl.he_mlp(widths, [98, sum(widths), 0])), wl.cube(widths[0])
    got = []
    for _ in range(5):
        cx = pcx.extract(m, box.lo, box.hi)
        got.append((*cx.copy(), cx.steps()))
        graph = cx.info().from_graph
        cx.close()
    assert graph == (0 if one_workgroup else 1)
    bt = pcx.Batch([m], [(box.lo, box.hi)])
    assert not one_workgroup or bt.stats().fallbacks == 0
    got.append((*bt.copy(0), bt.steps(0)))
    bt.close()
    m.close()
    for other in got[1:]:
        for a, b in zip(other, got[0]):
            assert a.shape == b.shape and np.array_equal(a, b)
