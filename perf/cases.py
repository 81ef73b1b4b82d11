"""The work that a user of this library has it do, as cases that can be timed.

Every case is one pass through the public Python entry points (``pcx``,
``torch_ops``) on a random-initialised network: He-normal weights, biases
uniform in (-0.5, 0.5), on a box (or a simplex), as in the paper's experiments
(Sec. 5.1.2) and this repository's workloads. Extracted complexes
are read as torch tensors over the library's own device arrays; the batched and
the served form hand their results over in host arrays, so there the copies
belong to the pass.
"""
from __future__ import annotations

import itertools
import math

import numpy as np
import torch

from paper_2306_07212_amd import pcx, torch_ops

DEV = "cuda:0"
EXACT_VERTICES = 1.5e6  # largest predicted complex that exact() builds in numpy


# ------------------------------------------------------------------- the cases

def listed():
    return [
        # the smallest call: one launch's latency and the host path around it
        {"name": "extract_2x8x8", "kind": "extract", "widths": "2-8-8-1", "output": False},
        # a small decision boundary in the plane (widths of the paper's bunny network)
        {"name": "extract_2x50x50_output", "kind": "extract", "widths": "2-50-50-1", "output": True},
        # an ordinary implicit surface: 0.7M vertices, and its zero level set
        {"name": "extract_3x64x3_output", "kind": "extract", "widths": "3-64-64-64-1", "output": True},
        # the largest: 768 neurons, 38M vertices
        {"name": "extract_3x256x3", "kind": "extract", "widths": "3-256-256-256-1", "output": False},
        # higher input dimension, on a simplex in place of the 2^D corners
        {"name": "simplex_6x32x32", "kind": "simplex", "widths": "6-32-32-1", "output": False},
        # only the zero level set is wanted: pruning during subdivision
        {"name": "levelset_3x64x3", "kind": "levelset", "widths": "3-64-64-64-1", "output": True},
        # into the caller's own buffers, for loops that may not allocate; ragged widths
        {"name": "into_2x61x47x33", "kind": "into", "widths": "2-61-47-33-1", "output": False},
        # one step of optimising a level set through its vertices (Sec. 5.3): forward, loss, backward
        {"name": "train_f64_3x64x3", "kind": "train", "widths": "3-64-64-64-1", "precision": "f64"},
        # the same with float32 parameters, smaller and ragged
        {"name": "train_f32_3x40x23", "kind": "train", "widths": "3-40-23-1", "precision": "f32"},
        # many small networks at once: 2 -> [w] x d -> 1, w in {8, 16, 32, 64}, d in {2, 3, 4}
        {"name": "batch_256", "kind": "batch", "n": 256},
        # a burst of requests to the server: D in {2, 3}, ragged widths, depth 2 to 4
        {"name": "serve_16", "kind": "serve", "n": 16, "widest": 32},
        # sign-vectors of every region of an extracted complex (one for about every vertex)
        {"name": "regions_3x64x64", "kind": "regions", "widths": "3-64-64-1", "output": False},
    ]


def draw(rng):
    kind = rng.choice(["extract", "extract", "extract", "simplex", "levelset", "into", "train", "batch", "serve",
                       "regions"])
    if kind == "batch":
        return {"kind": kind, "n": round(math.exp(rng.uniform(math.log(16), math.log(400))))}
    if kind == "serve":
        return {"kind": kind, "n": rng.randint(4, 20), "widest": rng.randint(20, 44)}
    # input dimensions and the range of complex sizes (vertices) of each path
    dims, small, large = {
        "extract": ([1, 2, 2, 3, 3, 3, 4, 5], 60, 1.5e7),
        "simplex": ([2, 3, 4, 6], 200, 5e6),
        "levelset": ([2, 3, 3, 4], 500, 1e6),
        "into": ([2, 3], 200, 1e5),
        "train": ([2, 3, 3], 500, 7e5),
        "regions": ([2, 3, 3, 4], 500, 3e5),
    }[kind]
    D = rng.choice(dims)
    large = min(large, {1: 300, 2: 2e5}.get(D, large))  # on the line and in the plane: hundreds of neurons
    target = math.exp(rng.uniform(math.log(small), math.log(large)))
    neurons = next(n for n in range(2 * D + 2, 2000) if n >= 768 or vertices_of(D, n) >= target)
    depth = rng.choice([1, 2, 2, 3, 3, 4])
    depth = max(-(-neurons // 256), min(depth, max(1, neurons // 4)))
    cuts = [rng.uniform(0.7, 1.3) for _ in range(depth)]
    hidden = [max(2, min(256, round(neurons * c / sum(cuts)))) for c in cuts]
    case = {"kind": kind, "widths": "-".join(str(w) for w in [D] + hidden + [1])}
    if kind == "train":
        case["precision"] = rng.choice(["f64", "f64", "f32"])
    else:
        case["output"] = kind == "levelset" or (kind != "regions" and rng.random() < 0.4)
    return case


def widths_of(case):
    return [int(w) for w in case["widths"].split("-")]


def vertices_of(D, n):
    """About how many vertices n neurons cut the cube (or a simplex) into (fitted on random networks)."""
    if D == 1:
        return 2.0 + 0.7 * n
    return 2.0 ** D + 2.0 * n + {2: 0.4, 3: 0.083, 4: 0.022}.get(D, 0.5 / math.factorial(D)) * float(n) ** D


def subdivided(case):
    """Widths of the layers whose neurons subdivide the domain."""
    w = widths_of(case)
    return w[1:] if case.get("output") or case["kind"] == "train" else w[1:-1]


# ------------------------------------------------------------ inputs and plans

def network(widths, seed):
    """(W, b, lo, hi, corners) of a network and its domain.

    The random-initialised network belongs to the widths; the seed draws one of its equivalent forms (the neurons of
    each layer in another order and on another scale, the input axes in another order, direction, scale and place).
    So every seed has other inputs and outputs, and a complex of the same size."""
    base = np.random.default_rng(widths)
    W, b = [], []
    for k, n in zip(widths[:-1], widths[1:]):
        W.append(base.standard_normal((n, k)) * np.sqrt(2.0 / k))
        b.append(base.uniform(-0.5, 0.5, n))
    rng, D = np.random.default_rng(seed), widths[0]
    for l, n in enumerate(widths[1:-1]):
        order, scale = rng.permutation(n), np.exp(rng.uniform(-0.3, 0.3, n))
        W[l], b[l] = W[l][order] * scale[:, None], b[l][order] * scale
        W[l + 1] = W[l + 1][:, order] / scale
    axes, side = rng.permutation(D), rng.choice([-1.0, 1.0], D) * np.exp(rng.uniform(-0.3, 0.3, D))
    centre = rng.uniform(-0.5, 0.5, D)
    W[0] = W[0][:, axes] / side
    b[0] = b[0] - W[0] @ centre
    # the corner simplex of the cube's volume
    unit = np.vstack([-np.ones(D), 2.0 * math.factorial(D) ** (1.0 / D) * np.eye(D) - 1.0])
    return W, b, centre - np.abs(side), centre + np.abs(side), centre + side * unit[:, axes]


def batch_widths(n, rng):
    return [[2] + [int(rng.choice([8, 16, 32, 64]))] * int(rng.choice([2, 3, 4])) + [1] for _ in range(n)]


def request_widths(n, widest, rng):
    return [[int(rng.choice([2, 3]))] + [int(rng.integers(16, widest + 1))] * int(rng.choice([2, 3, 4])) + [1]
            for _ in range(n)]


def members(case, seed):
    """(widths, (W, b, lo, hi, corners)) of every network of a batch or burst."""
    sizes = np.random.default_rng(case["n"])
    many = (batch_widths(case["n"], sizes) if case["kind"] == "batch"
            else request_widths(case["n"], case["widest"], sizes))
    return [(w, network(w, [seed, i])) for i, w in enumerate(many)]


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("batch", "serve"):
        nets = members(case, seed)
        mlps = [pcx.MLP(w, W, b) for w, (W, b, *_) in nets]
        boxes = [(lo, hi) for _, (_, _, lo, hi, _) in nets]
        state = {"kind": kind, "mlps": mlps, "boxes": boxes}
        if kind == "serve":
            state["server"] = pcx.Server()
        return state
    widths = widths_of(case)
    D = widths[0]
    W, b, lo, hi, corners = network(widths, seed)
    state = {"kind": kind, "widths": widths, "lo": lo, "hi": hi, "output": case.get("output", True)}
    if kind == "train":
        dtype = torch.float64 if case["precision"] == "f64" else torch.float32
        state["W"] = [torch.tensor(w, dtype=dtype, device=DEV, requires_grad=True) for w in W]
        state["b"] = [torch.tensor(x, dtype=dtype, device=DEV, requires_grad=True) for x in b]
        state["precision"] = case["precision"]
        return state
    state["mlp"] = pcx.MLP(widths, W, b)
    if kind == "simplex":
        state["corners"] = corners
    if kind == "regions":
        state["complex"] = pcx.extract(state["mlp"], state["lo"], state["hi"], include_output=state["output"])
    if kind == "into":
        words = 1 + sum(-(-n // 32) for n in subdivided(case))
        room = int(2.0 * vertices_of(D, sum(subdivided(case)))) + 256
        state["X"] = torch.empty((room, D), dtype=torch.float64, device=DEV)
        state["signs"] = torch.empty((room, words), dtype=torch.int64, device=DEV)
        state["edges"] = torch.empty((room * (D + 1), 2), dtype=torch.int32, device=DEV)
    return state


# ------------------------------------------------------------------- one pass

class DeviceArray:
    """A complex's device array for torch.as_tensor: the tensor keeps the complex alive."""

    def __init__(self, owner, pointer, shape, typestr):
        self.owner = owner
        self.__cuda_array_interface__ = {"data": (pointer, False), "shape": shape, "typestr": typestr, "version": 3}


def tensors_of(cx):
    info = cx.info()
    X, signs, edges = cx.device_pointers()
    return {"coords": torch.as_tensor(DeviceArray(cx, X, (info.V, info.D), "<f8"), device=DEV),
            "signs": torch.as_tensor(DeviceArray(cx, signs, (info.V, info.Wd), "<i8"), device=DEV),
            "edges": torch.as_tensor(DeviceArray(cx, edges, (info.E, 2), "<i4"), device=DEV)}


def joined(complexes):
    """Host complexes of many networks, laid end to end."""
    return {"coords": np.concatenate([x.ravel() for x, _, _ in complexes]),
            "signs": np.concatenate([s.ravel().view(np.int64) for _, s, _ in complexes]),
            "edges": np.concatenate([e for _, _, e in complexes])}


def run(state):
    kind = state["kind"]
    if kind == "batch":
        batch = pcx.Batch(state["mlps"], state["boxes"])
        return joined([batch.copy(i) for i in range(len(batch))])
    if kind == "serve":
        server = state["server"]
        tickets = [server.submit(m, lo, hi) for m, (lo, hi) in zip(state["mlps"], state["boxes"])]
        complexes = []
        for ticket in tickets:
            complexes.append(server.copy(ticket))
            server.release(ticket)
        return joined(complexes)
    if kind == "train":
        params = state["W"] + state["b"]
        X, signs, edges = torch_ops.extract_coords(state["W"], state["b"], state["lo"], state["hi"],
                                                   include_output=True, precision=state["precision"])
        loss = torch_ops.level_set_edge_loss(X, signs, edges, state["widths"])
        return {"loss": loss.detach(), "grads": torch.autograd.grad(loss, params)}
    if kind == "regions":
        return state["complex"].regions().view(np.int64)
    stream = torch.cuda.current_stream().cuda_stream
    if kind == "into":
        info, steps = pcx.extract_into(state["mlp"], state["lo"], state["hi"], state["X"].data_ptr(),
                                       state["signs"].data_ptr(), state["edges"].data_ptr(), len(state["X"]),
                                       len(state["edges"]), include_output=state["output"], stream=stream)
        return {"coords": state["X"][:info.V], "signs": state["signs"][:info.V], "edges": state["edges"][:info.E],
                "steps": steps}
    if kind == "simplex":
        return tensors_of(pcx.extract_simplex(state["mlp"], state["corners"], include_output=state["output"],
                                              stream=stream))
    return tensors_of(pcx.extract(state["mlp"], state["lo"], state["hi"], include_output=state["output"],
                                  prune=kind == "levelset", stream=stream))


# ------------------------------------------------------- what a pass cannot avoid

def work_of_network(D, hidden):
    """Bytes and FLOPs of extracting one complex: the network read, the complex written, each layer's
    pre-activations at the vertices that its start has, and each new vertex's interpolation."""
    bytes_, flops, n, k = 0.0, 0.0, 0, D
    for N in hidden:
        bytes_ += 8.0 * (N * k + N)
        flops += 2.0 * k * N * vertices_of(D, n)
        flops += 3.0 * (D + N) * (vertices_of(D, n + N) - vertices_of(D, n))
        n, k = n + N, N
    words = 1 + sum(-(-N // 32) for N in hidden)
    V = vertices_of(D, n)
    return bytes_ + V * (8.0 * D + 8.0 * words) + 8.0 * D * V, flops


def work(case):
    kind = case["kind"]
    if kind in ("batch", "serve"):
        each = [work_of_network(w[0], w[1:-1]) for w, _ in members(case, 0)]
        return {"bytes": sum(b for b, _ in each), "flops": sum(f for _, f in each)}
    D, hidden = widths_of(case)[0], subdivided(case)
    bytes_, flops = work_of_network(D, hidden)
    V, rows = vertices_of(D, sum(hidden)), 8.0 * (1 + sum(-(-N // 32) for N in hidden))
    if kind == "levelset":
        bytes_ *= 0.05  # about what pruning keeps
    if kind == "train":
        bytes_, flops = 2 * bytes_, 3 * flops
    if kind == "regions":
        bytes_, flops = 2 * V * rows + 8.0 * D * V, 0.0
    return {"bytes": bytes_, "flops": flops}


# --------------------------------------------------------------- in numpy alone

class Rows:
    """An array that grows at its end."""

    def __init__(self, a):
        self.room, self.n = a, len(a)

    @property
    def a(self):
        return self.room[:self.n]

    def add(self, more):
        need = self.n + len(more)
        if need > len(self.room):
            room = np.zeros((need + need // 2, *self.room.shape[1:]), self.room.dtype)
            room[:self.n] = self.a
            self.room = room
        self.room[self.n:need] = more
        self.n = need


class Plain:
    """Edge subdivision in numpy (float64): the five steps of Sec. 4.2, in the library's order of vertices
    (splitting edges in edge order) and edges (the second halves in edge order, then the intersecting edges by
    their 2-face's first appearance: splitting edges in order, each one's zeros in entry order, + before -)."""

    def __init__(self, W, b, lo, hi, corners, nsub, simplex=False, prune=False):
        D = len(lo)
        self.D, self.m = D, D + 1 if simplex else 2 * D
        if simplex:
            self.X = corners
            self.edges = np.array(list(itertools.combinations(range(D + 1), 2)), np.int64).reshape(-1, 2)
            dom = np.eye(D + 1, dtype=np.int8)
        else:
            ids = np.arange(1 << D)
            up = ((ids[:, None] >> np.arange(D)) & 1).astype(bool)
            self.X = np.where(up, hi, lo)
            self.edges = np.array([(c, c | 1 << j) for j in range(D) for c in range(1 << D) if not c >> j & 1])
            dom = np.empty((1 << D, 2 * D), np.int8)
            dom[:, 0::2], dom[:, 1::2] = up, ~up
        total = self.m + sum(len(x) for x in b[:nsub])
        S = np.zeros((len(self.X), total), np.int8)
        S[:, :self.m] = dom
        self.start, self.Z, self.steps = [], [], []  # the tape: vertices at each layer start, rows, steps
        self.keys = np.random.default_rng(7).integers(0, 1 << 63, (2, total), dtype=np.uint64)
        X, E, S, h, base = Rows(self.X), Rows(self.edges), Rows(S), self.X, self.m
        for l in range(nsub):
            z = h @ W[l].T + b[l]
            N = z.shape[1]
            if prune:
                later, hh = [np.sign(z)], z
                for q in range(l + 1, nsub):
                    hh = np.maximum(hh, 0.0) @ W[q].T + b[q]
                    later.append(np.sign(hh))
                later = np.concatenate(later, axis=1)
                keep = (later[E.a[:, 0]] != later[E.a[:, 1]]).any(axis=1)
                live = np.zeros(X.n, bool)
                live[E.a[keep].ravel()] = True
                number = np.cumsum(live) - 1
                X, E, S, z = Rows(X.a[live]), Rows(number[E.a[keep]]), Rows(S.a[live]), z[live]
            S.a[:, base:base + N] = np.sign(z)
            self.start.append(X.n)
            Z = Rows(z)
            for j in range(N):
                self._step(X, E, S, Z, j, base, N)
            self.Z.append(Z.a)
            h, base = np.maximum(Z.a, 0.0), base + N
        self.X, self.edges, self.S = X.a, E.a, S.a

    def _step(self, X, edges, signs, rows, j, base, N):
        E, S, z, V0, entry = edges.a, signs.a, rows.a, X.n, base + j
        sj = S[:, entry].copy()
        cut = np.flatnonzero(sj[E[:, 0]] * sj[E[:, 1]] < 0)
        n = len(cut)
        a, b = E[cut, 0], E[cut, 1]
        p, q = np.where(sj[a] > 0, a, b), np.where(sj[a] > 0, b, a)
        t = z[p, j] / (z[p, j] - z[q, j])
        x0 = V0 + np.arange(n)
        zn = z[p] + t[:, None] * (z[q] - z[p])
        zn[:, j] = 0.0
        face = np.where(S[a, :entry] != 0, S[a, :entry], S[b, :entry])
        Sn = np.zeros((n, S.shape[1]), np.int8)
        Sn[:, :entry] = face
        Sn[:, entry + 1:base + N] = np.sign(zn[:, j + 1:])
        E[cut, 1] = x0
        edges.add(np.stack([x0, b], axis=1))
        if self.D > 1 and n:
            plus, minus = self.keys[:, :entry]
            row = ((face > 0) * plus + (face < 0) * minus).sum(axis=1, dtype=np.uint64)
            s, e = np.nonzero(face == 0)
            twice = np.where(e < self.m, 1, 2)
            s, e = np.repeat(s, twice), np.repeat(e, twice)
            second = np.zeros(len(s), np.int64)
            second[1:] = (s[1:] == s[:-1]) & (e[1:] == e[:-1])
            order = np.argsort(row[s] + self.keys[second, e], kind="stable").reshape(-1, 2)  # each 2-face is met twice
            order = order[np.argsort(order[:, 0])]
            edges.add(V0 + s[order])
        X.add(X.a[p] + t[:, None] * (X.a[q] - X.a[p]))
        signs.add(Sn)
        rows.add(zn)
        self.steps.append((V0, p, q, j))


def packed(S, m, hidden):
    """Sign rows as 64-bit words, two bits an entry (01 +, 10 -), each layer from a fresh word."""
    codes = np.where(S > 0, 1, np.where(S < 0, 2, 0)).astype(np.uint64)
    words, at = [], 0
    for n in [m] + list(hidden):
        for w in range(0, n, 32):
            part = codes[:, at + w:at + min(w + 32, n)]
            words.append((part << (2 * np.arange(part.shape[1], dtype=np.uint64))).sum(axis=1, dtype=np.uint64))
        at += n
    return np.stack(words, axis=1).view(np.int64)


def plain_gradient(c, W, b):
    """Loss (summed squared lengths of the output's level-set edges) and its gradients, by hand in reverse."""
    on = c.S[:, -1 - (len(b[-1]) - 1)] == 0
    ls = c.edges[on[c.edges].all(axis=1)]
    d = c.X[ls[:, 0]] - c.X[ls[:, 1]]
    gx = np.zeros_like(c.X)
    np.add.at(gx, ls[:, 0], 2 * d)
    np.add.at(gx, ls[:, 1], -2 * d)
    gW, gb, gz = [None] * len(W), [None] * len(W), np.zeros_like(c.Z[-1])
    steps = list(c.steps)
    for l in reversed(range(len(W))):
        Z, Vs = c.Z[l], c.start[l]
        for _ in range(Z.shape[1]):
            V0, p, q, j = steps.pop()
            x0 = slice(V0, V0 + len(p))
            zp, zq = Z[p, j], Z[q, j]
            t, den = zp / (zp - zq), (zp - zq) ** 2
            g = gz[x0].copy()
            g[:, j] = 0.0
            gt = (gx[x0] * (c.X[q] - c.X[p])).sum(axis=1) + (g * (Z[q] - Z[p])).sum(axis=1)
            for v, share, slope in ((p, 1 - t, -zq / den), (q, t, zp / den)):
                np.add.at(gx, v, share[:, None] * gx[x0])
                np.add.at(gz, v, share[:, None] * g)
                np.add.at(gz, (v, j), gt * slope)
        h = c.X[:Vs] if l == 0 else np.maximum(c.Z[l - 1][:Vs], 0.0)
        gW[l], gb[l] = gz[:Vs].T @ h, gz[:Vs].sum(axis=0)
        if l:
            gz = (gz[:Vs] @ W[l]) * (c.Z[l - 1][:Vs] > 0)
    return (d * d).sum(), gW, gb


def plain_run(case, net):
    hidden = subdivided(case)
    c = Plain(*net, len(hidden), case["kind"] == "simplex", case["kind"] == "levelset")
    return c, {"coords": c.X, "signs": packed(c.S, c.m, hidden), "edges": c.edges.astype(np.int32)}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("batch", "regions"):
        return None  # hundreds of networks take longer; regions are whole numbers
    if kind == "serve":
        nets = members(case, seed)
        if sum(vertices_of(w[0], sum(w[1:-1])) for w, _ in nets) > EXACT_VERTICES:
            return None
        done = [plain_run({"kind": "extract", "widths": "-".join(map(str, w))}, net)[1] for w, net in nets]
        return joined([(o["coords"], o["signs"], o["edges"]) for o in done])
    widths = widths_of(case)
    if vertices_of(widths[0], sum(subdivided(case))) * len(subdivided(case)) > EXACT_VERTICES * 3:
        return None
    net = network(widths, seed)
    if kind == "train" and case["precision"] == "f32":
        net = tuple([x.astype(np.float32).astype(np.float64) for x in part] for part in net[:2]) + net[2:]
    c, out = plain_run(case, net)
    if kind == "into":
        out["steps"] = None
    if kind == "train":
        loss, gW, gb = plain_gradient(c, *net[:2])
        return {"loss": loss, "grads": tuple(gW + gb)}
    return out
