"""The backward's reverse pass by depth at every group width (16, 32 and 64
lanes, one, two and four columns a lane), over one to three layers: FP64
gradients against the implicit-function closed form on the oracle's complex,
FP32 against FP64, and the tape of a sort-paired extraction. Tolerances are
those of the full workload's tests (1e-8 relative; 1e-4 for FP32)."""
import numpy as np
import pytest

from implicit import implicit_grad, level_set_loss
from paper_2306_07212_amd import workloads as wl
from test_gpu_backward import gpu_grads, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("widths", [[2, 1, 1], [2, 16, 1], [2, 17, 33, 1], [2, 64, 9, 1], [2, 65, 1], [2, 129, 1],
                                    [2, 200, 20, 1], [3, 12, 9, 7, 1], [4, 9, 6, 1]])
def test_gradients_of_every_group_width(oracle_lib, widths):
    from paper_2306_07212_amd import torch_ops
    net, box = wl.he_mlp(widths, [94, sum(widths)]), wl.cube(widths[0])
    loss, gW, gb, V = gpu_grads(torch_ops, net)
    r = oracle_lib.extract(net, box.lo, box.hi, include_output=True)
    L, G, n = level_set_loss(r.X, r.S, r.edges, net.widths)
    print(f"[bwd] {widths}: {V} vertices, {n} level-set edges", flush=True)
    assert V == r.V
    assert abs(loss - L) <= 1e-9 * max(1.0, abs(L))
    if n == 0:  # the level set does not meet the box: no gradient
        assert all(np.all(g == 0.0) for g in gW + gb)
        return
    iW, ib = implicit_grad(net, box.lo, box.hi, r.X, r.S, G)
    assert rel(gW + gb, iW + ib) < 1e-8
    _, fW, fb, _ = gpu_grads(torch_ops, net, "f32")
    assert rel(fW + fb, gW + gb) < 1e-4


def test_tape_of_a_sort_paired_extraction_gives_the_same_gradients():
    import torch
    from paper_2306_07212_amd import pcx
    net, box = wl.he_mlp([3, 20, 14, 1], [94, 1]), wl.cube(3)
    m = pcx.MLP.from_net(net)
    got = []
    for pairing in ("hash", "sort"):
        cx = pcx.extract(m, box.lo, box.hi, include_output=True, record_tape=True, pairing=pairing)
        X, _, _ = cx.copy()
        # dL/dx from the coordinates alone: the two pairings number the edges apart, not the vertices' values
        order = np.lexsort(X.T)
        g = np.empty_like(X)
        g[order] = np.random.default_rng(3).standard_normal(X.shape)
        g = torch.from_numpy(g).cuda()
        gW = [torch.empty(w.shape, dtype=torch.float64, device="cuda") for w in net.W]
        gb = [torch.empty(x.shape, dtype=torch.float64, device="cuda") for x in net.b]
        pcx.backward(m, cx, g.data_ptr(), [t.data_ptr() for t in gW], [t.data_ptr() for t in gb], pcx.PCX_F64,
                     torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        got.append((np.sort(X, axis=0), [t.cpu().numpy() for t in gW + gb]))
        cx.close()
    m.close()
    assert np.allclose(got[0][0], got[1][0], rtol=0, atol=1e-12)
    assert rel(got[0][1], got[1][1]) < 1e-8
