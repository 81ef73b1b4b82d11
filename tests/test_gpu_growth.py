"""First extractions of large networks, several at a time on streams of their
own while the host is slow to follow: steps that find the storage too small are
redone, and every complex is the one extracted alone."""
import threading

import numpy as np
import pytest

from paper_2306_07212_amd import workloads as wl

pytestmark = pytest.mark.gpu

WIDTHS = [[3, 75, 75, 75, 1], [3, 120, 120, 1], [3, 100, 100, 1], [2, 250, 250, 1]]


def test_storage_grown_while_other_extractions_run():
    import torch
    from paper_2306_07212_amd import pcx
    nets = [wl.he_mlp(w, [101, sum(w)]) for w in WIDTHS]
    bad = []

    def one(net):
        m, box = pcx.MLP.from_net(net), wl.cube(net.D)
        st = torch.cuda.Stream()
        cx = pcx.extract(m, box.lo, box.hi, stream=st.cuda_stream)
        got = (cx.info().V, cx.info().E, cx.steps())
        cx.close()
        m.close()
        return got

    want = [one(n) for n in nets]

    def work(i):
        for r in range(10):
            try:
                got = one(nets[i])
            except RuntimeError as e:
                bad.append((WIDTHS[i], r, str(e)))
                return
            if got[:2] != want[i][:2] or not np.array_equal(got[2], want[i][2]):
                bad.append((WIDTHS[i], r, got[:2], want[i][:2]))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(nets))]
    for t in threads:
        t.start()
    while any(t.is_alive() for t in threads):  # (the host's other threads want its cores and the lock)
        sum(range(20000))
    assert not bad, bad


def test_steps_redone_in_grown_storage_while_other_extractions_run(monkeypatch, capfd):
    """The same four networks from the smallest storage (every extraction grows it and redoes the steps that found it
    too small: the library's own count says so), several at a time."""
    import re
    import torch
    from paper_2306_07212_amd import pcx
    nets = [wl.he_mlp(w, [101, sum(w)]) for w in WIDTHS]
    bad = []

    def one(net):
        m, box = pcx.MLP.from_net(net), wl.cube(net.D)
        st = torch.cuda.Stream()
        cx = pcx.extract(m, box.lo, box.hi, stream=st.cuda_stream)
        got = (cx.info().V, cx.info().E, cx.steps())
        cx.close()
        m.close()
        return got

    want = [one(n) for n in nets]
    monkeypatch.setenv("PCX_SMALL_START", "1")
    monkeypatch.setenv("PCX_VERBOSE", "1")
    capfd.readouterr()

    def work(i):
        for r in range(4):
            try:
                got = one(nets[i])
            except RuntimeError as e:
                bad.append((WIDTHS[i], r, str(e)))
                return
            if got[:2] != want[i][:2] or not np.array_equal(got[2], want[i][2]):
                bad.append((WIDTHS[i], r, got[:2], want[i][:2]))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(nets))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    redone = [int(x) for x in re.findall(r"redone after growing the storage: (\d+)", capfd.readouterr().err)]
    assert not bad, bad
    print(f"[growth] steps redone: {redone}", flush=True)
    assert len(redone) == 4 * len(nets) and min(redone) > 0
