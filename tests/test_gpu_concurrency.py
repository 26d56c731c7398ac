"""Reentrancy per stream: bta_selinv (which leases helper streams and events
for its preprocessing and copy-outs) called from two host threads at once,
each on its own stream with its own workspace and outputs, several times in a
row; both results compared block by block with the oracle."""
import threading

import numpy as np
import pytest

import oracle
from paper_2503_17528_amd import synth
from tests.gpu_util import TOL, errs, say, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("least", [False, True])
def test_selinv_threads_either_sweep(least):
    """The same threads and streams at sizes of both sweeps: with the least
    workspace, where the blocks are swept product by product on leased streams, and
    with the whole one, where two persistent sweeps share the chip; larger blocks
    beside them, which have no other way."""
    _run_threads([(12, 192, 5), (9, 257, 3), (3, 1282, 4), (8, 512, 70)], least)


def _run_threads(shapes, least):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2503_17528_amd import bta

    bta.lib()
    say(f"case concurrency: selinv on {len(shapes)} threads, shapes {shapes}, least workspace {least}")
    size = bta.bta_workspace_min_bytes if least else bta.bta_workspace_bytes
    ref, Ls, outs, works = [], [], [], []
    for k, s in enumerate(shapes):
        Q = synth.make_np(synth.workload(*s, "literal" if s[1] <= 512 else "scaled"), 40 + k)
        F = oracle.pobtaf(Q["D"], Q["B"], Q["R"], Q["T"])
        Xo = oracle.pobtasi(F["LD"], F["LB"], F["LR"], F["LT"])
        ref.append({"D": Xo["XD"], "B": Xo["XB"], "R": Xo["XR"], "T": Xo["XT"]})
        Ls.append(to_dev({x: F["L" + x] for x in "DBRT"}))
        outs.append([tuple(torch.empty_like(t) for t in Ls[k]) for _ in range(4)])
        works.append(torch.empty(size(bta.BTA_OP_SELINV, *s), dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in shapes]
    start = threading.Barrier(len(shapes))
    failures = []

    def run(k):
        try:
            start.wait()
            for out in outs[k]:
                with torch.cuda.stream(streams[k]):
                    bta.selinv(*Ls[k], out=out, work=works[k], stream=streams[k])
        except Exception as e:  # reported below, on the main thread
            failures.append((k, repr(e)))

    threads = [threading.Thread(target=run, args=(k,)) for k in range(len(shapes))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not failures, failures
    for k, s in enumerate(shapes):
        e = errs(dict(zip("DBRT", to_np(outs[k][0]))), ref[k], lower=())
        say(f"   thread {k} {s}: {e}")
        assert max(e.values()) < TOL, e
        for out in outs[k][1:]:
            assert all(torch.equal(x, y) for x, y in zip(outs[k][0], out))


def test_selinv_two_threads_two_streams():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2503_17528_amd import bta

    bta.lib()
    shapes = [(12, 192, 5), (9, 256, 3)]
    say(f"case concurrency: selinv on two threads and two streams, shapes {shapes}")
    ref, Ls, outs, works = [], [], [], []
    for k, s in enumerate(shapes):
        wl = synth.workload(*s)
        Q = synth.make_np(wl, 40 + k)
        F = oracle.pobtaf(Q["D"], Q["B"], Q["R"], Q["T"])
        Xo = oracle.pobtasi(F["LD"], F["LB"], F["LR"], F["LT"])
        ref.append({"D": Xo["XD"], "B": Xo["XB"], "R": Xo["XR"], "T": Xo["XT"]})
        D, B, R, T = (torch.from_numpy(Q[x]).to("cuda") for x in "DBRT")
        L = bta.factor(D, B, R, T)[:4]
        Ls.append(L)
        outs.append(tuple(torch.empty_like(t) for t in L))
        works.append(bta.workspace(bta.BTA_OP_SELINV, *s, "cuda")[0])
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    start = threading.Barrier(2)
    failures = []

    def run(k):
        try:
            start.wait()
            for _ in range(4):
                with torch.cuda.stream(streams[k]):
                    bta.selinv(*Ls[k], out=outs[k], work=works[k], stream=streams[k])
        except Exception as e:  # reported below, on the main thread
            failures.append((k, repr(e)))

    threads = [threading.Thread(target=run, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not failures, failures
    for k in range(2):
        e = errs(dict(zip("DBRT", to_np(outs[k]))), ref[k], lower=())
        say(f"   thread {k} {shapes[k]}: {e}")
        assert max(e.values()) < TOL, e
