"""Steps of more than 16384 key slots count their slots' records instead of
reading every partner's: with few enough hash bits that some of such a step's
2-faces share a word, it still goes to the exact pass, and the complex is the
one without collisions, bit for bit."""
import numpy as np
import pytest

from paper_2306_07212_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("widths", [[3, 80, 60, 1], [5, 16, 14, 1]])
@pytest.mark.parametrize("bits", [34, 38, 42])
def test_collisions_in_large_steps(monkeypatch, widths, bits):
    from paper_2306_07212_amd import pcx
    m, box = pcx.MLP.from_net(wl.he_mlp(widths, [99, sum(widths)])), wl.cube(widths[0])
    monkeypatch.setenv("PCX_NO_TINY", "1")
    got = []
    for hook in (None, str(bits)):
        if hook:
            monkeypatch.setenv("PCX_DEBUG_HASH_BITS", hook)
        cx = pcx.extract(m, box.lo, box.hi)
        got.append((*cx.copy(), cx.steps()))
        exact = cx.info().exact_steps
        cx.close()
    m.close()
    large = int((got[0][3][:, 3] * 2 > 16384).sum())
    print(f"[pair count] {widths} {bits} bits: {exact} steps by the exact pass, {large} large ones", flush=True)
    assert large > 0 and (bits > 34 or exact > 0)
    for a, b in zip(*got):
        assert a.shape == b.shape and np.array_equal(a, b)
