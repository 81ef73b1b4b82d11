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


@pytest.mark.parametrize("full_grids", ["1", "0"])
@pytest.mark.parametrize("widths,bits", [([3, 40, 30, 1], 2), ([4, 12, 9, 1], 2), ([2, 60, 50, 1], 2),
                                         ([3, 80, 60, 1], 12), ([5, 16, 14, 1], 12)])
def test_every_crowded_step_is_found(monkeypatch, capfd, widths, bits, full_grids):
    """Hashes of b <= 24 bits leave all of a step's faces one table key and 2^b words to start their probes at, so of
    more than 2^b faces two meet for certain, and such a step must fail the look at its records, whichever launch
    takes it: with the largest grids every step counts them in a launch of its own, else those of more than 16384
    slots do (with 12 bits there are some, and none of them is small). The library names the steps."""
    import re
    from paper_2306_07212_amd import pcx
    m, box = pcx.MLP.from_net(wl.he_mlp(widths, [99, sum(widths)])), wl.cube(widths[0])
    monkeypatch.setenv("PCX_NO_TINY", "1")
    monkeypatch.setenv("PCX_FULL_GRIDS", full_grids)
    monkeypatch.setenv("PCX_VERBOSE", "1")
    got = []
    for hook in (None, str(bits)):
        if hook:
            monkeypatch.setenv("PCX_DEBUG_HASH_BITS", hook)
        capfd.readouterr()
        cx = pcx.extract(m, box.lo, box.hi)
        got.append((*cx.copy(), cx.steps()))
        cx.close()
        exact = {int(x) for x in re.findall(r"step (\d+) paired by the exact pass", capfd.readouterr().err)}
    m.close()
    keys = got[0][3][:, 3]  # two a face
    crowded = set(np.flatnonzero(keys // 2 > 2**bits).tolist())
    print(f"[pair count] {widths} {bits} bits: {len(exact)} steps by the exact pass, {len(crowded)} of more than "
          f"{2**bits} faces, {int((keys > 16384).sum())} of more than 16384 keys", flush=True)
    assert crowded and crowded <= exact
    assert bits == 2 or np.all(keys[sorted(crowded)] > 8192) and int((keys > 16384).sum()) > 0
    for a, b in zip(*got):
        assert a.shape == b.shape and np.array_equal(a, b)
