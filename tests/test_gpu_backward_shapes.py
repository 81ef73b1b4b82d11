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


def _reverse_on_the_line(w, b, grad, lo, hi, fused):
    """dL/db and dL/dw of a one-layer network on [lo, hi] in FP32 by the same sums: every vertex takes its children
    from the youngest on, one term each, fused (one rounding) or not; a term's product is exact in FP64."""
    N, f4 = len(w), np.float32
    G = 16 if N <= 16 else 32 if N <= 32 else 64

    def mac(a, x, acc):
        p = np.float64(f4(a)) * np.float64(f4(x))
        return f4(p + np.float64(acc)) if fused else f4(f4(p) + f4(acc))

    X, Z, par, neuron = [lo, hi], [w * lo + b, w * hi + b], [None, None], [-1, -1]
    line = [0, 1]  # vertices along the line
    for j in range(N):
        for i in range(len(line) - 1):
            p, q = line[i], line[i + 1]
            if (Z[p][j] > 0) == (Z[q][j] > 0):
                continue
            if Z[p][j] < 0:
                p, q = q, p  # p = V+
            t = Z[p][j] / (Z[p][j] - Z[q][j])
            z = Z[p] + t * (Z[q] - Z[p])
            z[j] = 0.0
            X.append(X[p] + t * (X[q] - X[p]))
            Z.append(z)
            par.append((p, q, t))
            neuron.append(j)
            line.insert(i + 1, len(X) - 1)
            break
    V = len(X)
    gx, gz = grad[:V].astype(f4), np.zeros((V, N), f4)
    kids, rec = [[] for _ in range(V)], [None] * V
    for v in range(2, V):
        kids[par[v][0]].append((v, 0))
        kids[par[v][1]].append((v, 1))
    for v in range(V - 1, -1, -1):
        for c, side in reversed(kids[v]):
            t, gt, fs = rec[c]
            s = f4(t) if side else f4(1.0 - t)
            gx[v] = mac(s, gx[c], gx[v])
            for k in range(N):
                own = k == neuron[c]
                gz[v, k] = mac(fs[side] if own else s, gt if own else gz[c, k], gz[v, k])
        if v < 2:
            continue
        p, q, t = par[v]
        lanes = np.zeros(G, f4)
        lanes[0] = mac(gx[v], X[q] - X[p], f4(0))
        for k in range(N):
            if k != neuron[v]:
                lanes[k] = mac(gz[v, k], Z[q][k] - Z[p][k], lanes[k])
        o = G // 2
        while o:
            lanes = lanes + lanes[np.arange(G) ^ o]
            o //= 2
        zp, zq = Z[p][neuron[v]], Z[q][neuron[v]]
        inv = 1.0 / ((zp - zq) * (zp - zq))
        rec[v] = (t, lanes[0], (f4(-zq * inv), f4(zp * inv)))
    return np.array([f4(gz[0, k] + gz[1, k]) for k in range(N)]), V


@pytest.mark.parametrize("N", [16, 32, 64])
def test_fp32_sums_round_once_a_term(N):
    """On the line every value of the FP32 reverse pass can be followed on the host. With fused terms the library's
    gradients are those bits (all but the few where FP64 stands in for the fused operation or a stored value differs
    in its last place); sums whose products are rounded by themselves agree in far fewer entries."""
    import torch
    from paper_2306_07212_amd import pcx
    same = {True: 0, False: 0}
    total = 0
    for seed in range(8):
        net, box = wl.he_mlp([1, N, 1], [95, N, seed]), wl.cube(1)
        m = pcx.MLP.from_net(net)
        cx = pcx.extract(m, box.lo, box.hi, record_tape=True)
        V = cx.info().V
        grad = np.random.default_rng([96, seed]).standard_normal(V)
        g = torch.from_numpy(grad).cuda()
        gW = [torch.empty(w.shape, dtype=torch.float64, device="cuda") for w in net.W]
        gb = [torch.empty(x.shape, dtype=torch.float64, device="cuda") for x in net.b]
        pcx.backward(m, cx, g.data_ptr(), [t.data_ptr() for t in gW], [t.data_ptr() for t in gb], pcx.PCX_F32,
                     torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        got = gb[0].cpu().numpy()
        cx.close()
        m.close()
        for fused in same:
            want, n = _reverse_on_the_line(net.W[0][:, 0], net.b[0], grad, float(box.lo[0]), float(box.hi[0]), fused)
            assert n == V
            live = want != 0.0
            same[fused] += int((got[live] == want[live]).sum())
            total += int(live.sum()) if fused else 0
    print(f"[bwd] 1-{N}-1: {same[True]} of {total} entries as with fused terms, {same[False]} without", flush=True)
    assert total > 4 * N and same[True] >= 0.98 * total
    assert same[False] < 0.8 * total  # (the two can be told apart)


@pytest.mark.parametrize("precision,size", [("PCX_F64", 8), ("PCX_F32", 4)])
def test_backward_holds_the_rows_of_two_layers(precision, size):
    """Device memory of one backward of a network of many layers: the rows of two layers, the coordinates' gradients,
    56 bytes per new vertex and 16 per vertex, and the partial sums (one layer's). Every block is rounded up to a
    MiB; the library keeps them in its pool, so what the call took is what is missing after it."""
    import torch
    from paper_2306_07212_amd import pcx
    net, box = wl.he_mlp([3, 64, 2, 2, 2, 2, 2, 2, 1], [97, 8]), wl.cube(3)
    m = pcx.MLP.from_net(net)
    cx = pcx.extract(m, box.lo, box.hi, include_output=True, record_tape=True)
    V = cx.info().V
    ZS, n = 64, V - int(cx.steps()[0, 0])
    rng = np.random.default_rng(98)
    g = torch.from_numpy(rng.standard_normal((V, 3))).cuda()
    gW = [torch.empty(w.shape, dtype=torch.float64, device="cuda") for w in net.W]
    gb = [torch.empty(x.shape, dtype=torch.float64, device="cuda") for x in net.b]
    torch.cuda.synchronize()
    pcx.cache_trim()
    before = torch.cuda.mem_get_info()[0]
    pcx.backward(m, cx, g.data_ptr(), [t.data_ptr() for t in gW], [t.data_ptr() for t in gb], getattr(pcx, precision),
                 torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    held = before - torch.cuda.mem_get_info()[0]
    pcx.cache_trim()
    part = 1024 * 64 * 65 * 8  # (at most 1024 chunks of a layer's entries)
    rows = V * ZS * size
    room = 2 * rows + V * 3 * size + 56 * n + 16 * V + part + 16 * (2 << 20)
    print(f"[bwd] {V} vertices, {precision}: {held / 2**20:.0f} MiB held, {room / 2**20:.0f} allowed, a layer's rows "
          f"{rows / 2**20:.0f}", flush=True)
    assert held <= room
    cx.close()
    m.close()
