"""Regions of rows longer than one group of lanes (17 and 33 words: 32 and 64
lanes a cell) and of every length modulo the 64 bits of a sort key: sorted,
distinct, as many as Euler's formula says, and holding the sign-vector of
random points of the box."""
import numpy as np
import pytest

from checks import unpack_signs
from paper_2306_07212_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("widths", [[2, 3, 1], [2, 33, 1], [2, 31, 33, 2, 1], [1, 40, 30, 1], [2, 230, 250, 1],
                                    [2, 226, 225, 230, 227, 1]])
def test_regions_are_sorted_distinct_and_complete(widths):
    from paper_2306_07212_amd import pcx
    net, box = wl.he_mlp(widths, [95, sum(widths)]), wl.cube(widths[0])
    m = pcx.MLP.from_net(net)
    cx = pcx.extract(m, box.lo, box.hi)
    info, rows = cx.info(), cx.regions()
    cx.close()
    m.close()
    D = widths[0]
    print(f"[regions] {widths}: {len(rows)} regions of {rows.shape[1]} words", flush=True)
    assert len(rows) == (info.E if D == 1 else 1 - info.V + info.E)
    order = np.lexsort(rows.T[::-1])
    assert np.array_equal(order, np.arange(len(rows))), "rows not in lexicographic order"
    assert (rows[1:] != rows[:-1]).any(axis=1).all(), "a region twice"
    have = {r.tobytes() for r in unpack_signs(rows, widths)[:, 2 * D:]}
    h, signs = np.random.default_rng(5).uniform(-1, 1, (500, D)), []
    for l in range(len(widths) - 2):
        z = h @ net.W[l].T + net.b[l]
        signs.append(np.sign(z).astype(np.int8))
        h = np.maximum(z, 0.0)
    for s in np.concatenate(signs, axis=1):
        assert s.tobytes() in have
