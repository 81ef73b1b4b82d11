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


def test_regions_in_pieces_hold_the_rows_once():
    """Rows of several pieces of the copy to the host: sorted and distinct, and beside what counting them takes the call
    holds them once, eight bytes a row for their order and a piece (every block rounded up to a MiB; the library
    keeps them in its pool, so what a call took is what is missing after it)."""
    import ctypes as C
    import torch
    from paper_2306_07212_amd import pcx
    m, box = pcx.MLP.from_net(wl.he_mlp([2, 226, 225, 230, 227, 1], [95, 908])), wl.cube(2)
    cx = pcx.extract(m, box.lo, box.hi)
    held, n = [], C.c_int64()
    for full in (False, True):
        pcx.cache_trim()
        before = torch.cuda.mem_get_info()[0]
        if full:
            rows = np.zeros((n.value, cx.info().Wd), np.uint64)
            rc = pcx._lib.pcx_regions(cx._h, rows.ctypes.data, C.byref(n), None)
        else:
            rc = pcx._lib.pcx_regions(cx._h, None, C.byref(n), None)
        assert rc == 0
        held.append(before - torch.cuda.mem_get_info()[0])
    cx.close()
    m.close()
    room = rows.nbytes + 8 * len(rows) + (16 << 20) + 8 * (2 << 20)
    print(f"[regions] {len(rows)} rows, {rows.nbytes / 2**20:.0f} MiB: {(held[1] - held[0]) / 2**20:.0f} MiB beside the "
          f"count's {held[0] / 2**20:.0f}, {room / 2**20:.0f} allowed", flush=True)
    assert rows.nbytes > 2 * (16 << 20) and held[1] - held[0] <= room
    order = np.lexsort(rows.T[::-1])
    assert np.array_equal(order, np.arange(len(rows)))
    assert (rows[1:] != rows[:-1]).any(axis=1).all()
