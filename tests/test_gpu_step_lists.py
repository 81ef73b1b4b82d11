"""The split lists that a step's pairing writes for the next neuron: chunks of
the scan and of the emission, with the owners counted in the emission (small
steps) or by a first launch (large ones), against the batched kernel's one list
and the two-pass compaction of redone steps. Every form must give the same
bits, and the oracle's complex."""
import numpy as np
import pytest

from checks import assert_same_complex, unpack_signs
from paper_2306_07212_amd import workloads as wl

pytestmark = pytest.mark.gpu

# widths, whether the oracle takes part: no key slots (D = 1), steps of a few
# slots, ragged layers, an edge count far above one scan tile, steps of more
# than 2048 lists' worth of slots and of both sides of 16384 key slots (D = 4)
CASES = [([1, 40, 17, 1], True), ([2, 5, 1], True), ([2, 130, 31, 1], True), ([3, 33, 27, 1], True),
         ([3, 200, 1], False), ([4, 26, 14, 1], False)]


@pytest.mark.parametrize("widths,oracle_too", CASES)
def test_every_form_of_the_split_list_gives_the_same_complex(oracle_lib, monkeypatch, widths, oracle_too):
    from paper_2306_07212_amd import pcx
    monkeypatch.setenv("PCX_NO_TINY", "1")
    net, box = wl.he_mlp(widths, [91, len(widths)]), wl.cube(widths[0])
    runs = {}
    for form, env in (("default", {}), ("largest grids", {"PCX_FULL_GRIDS": "1"}), ("grown", {"PCX_SMALL_START": "1"})):
        with monkeypatch.context() as mp:
            for k, v in env.items():
                mp.setenv(k, v)
            m = pcx.MLP.from_net(net)  # (a new handle: no sizes known from before)
            cx = pcx.extract(m, box.lo, box.hi)
            runs[form] = (*cx.copy(), cx.steps())
            cx.close()
            if form == "default":  # the known sizes, and the captured graph from the third request
                for again in ("second", "third", "fourth"):
                    cx = pcx.extract(m, box.lo, box.hi)
                    runs[again] = (*cx.copy(), cx.steps())
                    cx.close()
            m.close()
    m = pcx.MLP.from_net(net)
    bt = pcx.Batch([m], [(box.lo, box.hi)])
    runs["batched"] = (*bt.copy(0), bt.steps(0))
    bt.close()
    m.close()
    ref = runs["default"]
    for form, got in runs.items():
        for a, b in zip(got, ref):
            assert a.shape == b.shape and np.array_equal(a, b), f"{widths} {form}"
    if oracle_too:
        r = oracle_lib.extract(net, box.lo, box.hi)
        X, SG, Ed, steps = ref
        assert np.array_equal(steps, r.steps)
        assert_same_complex((X, unpack_signs(SG, net.widths), Ed), (r.X, r.S, r.edges))


@pytest.mark.parametrize("widths,batched", [(w, w != [3, 200, 1]) for w, _ in CASES])
def test_which_of_the_networks_the_batched_kernel_serves(widths, batched):
    """The batched form above is the one-workgroup kernels' own for every network but 3-200-1, whose prediction is
    above what a batch takes: nothing else falls back to the per-step path."""
    from paper_2306_07212_amd import pcx
    m, box = pcx.MLP.from_net(wl.he_mlp(widths, [91, len(widths)])), wl.cube(widths[0])
    bt = pcx.Batch([m], [(box.lo, box.hi)])
    st = bt.stats()
    assert st.fallbacks == (0 if batched else 1), st
    bt.close()
    m.close()
