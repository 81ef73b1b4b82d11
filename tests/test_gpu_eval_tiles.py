"""The per-step evaluation on the matrix cores at the edges of its tiles (32
rows, column blocks of 32 and 64, inputs staged 144 columns at a time) and with
its rows in spatial order: every sign entry of every vertex against a plain
FP64 forward pass of torch at the vertex's coordinates. Entries are compared
where |z| > 1e-9, and are below it where the sign-vector holds a zero (the
bounds of the oracle's own invariants)."""
import numpy as np
import pytest

from checks import unpack_signs
from paper_2306_07212_amd import workloads as wl

pytestmark = pytest.mark.gpu

# layer widths around 32, 64 and 128 columns; more than 144 inputs at once (a
# plane's few rows share few dead neurons: two rounds of staging); 0.2M rows
# in spatial order with odd widths on either side of the 128-column form; a
# narrow layer after a wide one and the other way round
SHAPES = [[2, 9, 33, 32, 1], [2, 64, 65, 31, 1], [2, 127, 128, 1], [2, 256, 255, 1], [2, 256, 12, 1], [2, 12, 200, 1],
          [3, 131, 129, 1], [3, 145, 101, 1], [5, 17, 10, 1]]


@pytest.mark.parametrize("widths", SHAPES)
def test_signs_are_the_forward_pass(monkeypatch, widths):
    import torch
    from paper_2306_07212_amd import pcx
    monkeypatch.setenv("PCX_NO_TINY", "1")
    net, box = wl.he_mlp(widths, [92, sum(widths)]), wl.cube(widths[0])
    m = pcx.MLP.from_net(net)
    cx = pcx.extract(m, box.lo, box.hi)
    X, SG, _ = cx.copy()
    cx.close()
    m.close()
    D, step = widths[0], 200000
    print(f"[eval] {widths}: {len(X)} vertices", flush=True)
    for v0 in range(0, len(X), step):
        S = torch.from_numpy(unpack_signs(SG[v0:v0 + step], widths)).cuda()
        h, at = torch.from_numpy(X[v0:v0 + step]).cuda(), 2 * D
        for l in range(len(widths) - 2):
            z = h @ torch.from_numpy(net.W[l]).cuda().T.contiguous() + torch.from_numpy(net.b[l]).cuda()
            s = S[:, at:at + widths[l + 1]]
            assert not bool(((z.abs() > 1e-9) & (torch.sign(z) != s)).any()), f"{widths} layer {l + 1}"
            assert not bool(((s == 0) & (z.abs() > 1e-9)).any()), f"{widths} layer {l + 1}: zeros"
            h, at = z.clamp(min=0.0), at + widths[l + 1]
