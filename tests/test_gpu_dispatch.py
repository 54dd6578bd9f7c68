"""Branches of the launch code that only large boxes, mixed batches or a
capturing caller reach.

* Streaming steps of 2D boxes whose rows start inside cache lines, and of
  batches that hold such a box: each case asserts that its step moves more
  than the memory-side cache and that its rows are off the lines. Boxes
  against the oracle with the method's bars (FP64 1e-10, FP32 1e-5), and
  against a small box that they repeat, bit for bit; batches against single
  contexts, FP64 1e-13 (sums in another order of the compiler's), others the
  method's bars (16-bit storage C 10 u_s and u 50 u_s).
* Long ddcc_step calls on a stream that the caller is capturing.
* Adjoint sweeps of boxes whose fields are recomputed for fewer than eight
  states at a time: a small box repeated periodically, against the small box.
"""
import numpy as np
import pytest

from paper_2311_10314_amd import workloads as W
from tests.helpers import oracle_run, rel_linf

pytestmark = pytest.mark.gpu

BAR = {"fp64": (1e-10, 1e-10), "fp32": (1e-5, 1e-5),
       "fp16": (10 * 2.0 ** -11, 50 * 2.0 ** -11),
       "bf16": (10 * 2.0 ** -8, 50 * 2.0 ** -8)}
CACHE = 256 << 20


def _step_bytes(nodes, N, precision):
    """Bytes that one 2D step moves: moving populations, float64 rest
    populations, flow set, T and history, each read and written."""
    pop = {"fp64": 8, "fp32": 4}.get(precision, 2)
    field = 8 if precision == "fp64" else 4
    return 2 * nodes * (N * 8 * pop + N * 8 + 9 * pop + field
                        + (2 * N + 4) * field)


def _off_lines(nx, precision):
    pop = {"fp64": 8, "fp32": 4}.get(precision, 2)
    return nx * pop % (32 if pop == 8 else 64) != 0


def _rep(v, copies):
    return np.tile(v, (1,) * (np.ndim(v) - 2) + copies)


def _repeated(wl, copies):
    return W.Workload("repeated", 2,
                      tuple(a * b for a, b in zip(wl.shape, copies)),
                      wl.lattice_f, wl.lattice_g, wl.params,
                      _rep(wl.psi, copies), _rep(wl.cos_theta_iN, copies),
                      _rep(wl.C0, copies), _rep(wl.u0, copies),
                      _rep(wl.P0, copies), 0)


@pytest.mark.parametrize("N,shape,precision", [
    (2, (830, 1001), "fp64"), (4, (561, 570), "fp64"), (2, (1001, 999), "fp32"),
    (3, (901, 901), "fp32")])
def test_streaming_steps_of_rows_off_lines(N, shape, precision):
    from paper_2311_10314_amd.ddcc import Sim
    assert _step_bytes(shape[0] * shape[1], N, precision) > CACHE
    assert _off_lines(shape[1], precision)
    print(shape, N, precision, flush=True)
    wl = W.random_small(2, N, shape, seed=61)
    sim = Sim.from_workload(wl, precision)
    sim.step(2)
    C, u, _ = sim.read_moments()
    sim.close()
    o = oracle_run(wl, 2)
    eC = max(rel_linf(C[i], o["C"][i]) for i in range(N))
    eu = rel_linf(u, o["u"])
    print("C %.2e u %.2e" % (eC, eu), flush=True)
    assert eC < BAR[precision][0] and eu < BAR[precision][1]


@pytest.mark.parametrize("N,small,copies,precision", [
    (4, (77, 111), (13, 9), "fp16"), (2, (109, 105), (11, 11), "bf16"),
    (3, (53, 85), (17, 11), "fp32")])
def test_streaming_steps_of_rows_off_lines_repeat(N, small, copies, precision):
    """A small box, whose steps stay in the cache, repeated until they do not:
    every node goes through the same arithmetic, so the moments repeat bit for
    bit."""
    from paper_2311_10314_amd.ddcc import Sim
    shape = tuple(a * b for a, b in zip(small, copies))
    assert _step_bytes(shape[0] * shape[1], N, precision) > CACHE
    assert _off_lines(shape[1], precision)
    wl = W.random_small(2, N, small, seed=66)
    out = []
    for w in (wl, _repeated(wl, copies)):
        print(w.shape, N, precision, flush=True)
        s = Sim.from_workload(w, precision)
        s.step(3)
        out.append(s.read_moments())
        s.close()
    for a, b in zip(*out):
        assert np.array_equal(_rep(a, copies), b)


@pytest.mark.parametrize("N,precision,tile,shapes", [
    (2, "fp32", 0, [(601, 560), (553, 601), (700, 333)]),
    (3, "fp64", 0, [(320, 640), (401, 390), (130, 66)]),
    (2, "fp16", 16, [(900, 640), (640, 901), (301, 600), (70, 96)]),
    (2, "bf16", 4, [(640, 1280), (640, 701), (301, 332)])])
def test_streaming_batches_with_rows_off_lines(N, precision, tile, shapes):
    from paper_2311_10314_amd.ddcc import Batch, Sim
    assert _step_bytes(sum(a * b for a, b in shapes), N, precision) > CACHE
    assert any(_off_lines(s[1], precision) for s in shapes)
    wls = [W.random_small(2, N, s, seed=62 + i) for i, s in enumerate(shapes)]
    print(shapes, N, precision, flush=True)
    b = Batch.from_workloads(wls, precision)
    if tile:
        b.set_tile(tile)
    b.set_graph(2)
    b.step(5)
    bar = (1e-13, 1e-13) if precision == "fp64" else BAR[precision]
    for i, wl in enumerate(wls):
        s = Sim.from_workload(wl, precision)
        s.step(5)
        C, u, _ = b.read_moments(i)
        Cs, us, _ = s.read_moments()
        s.close()
        eC = max(rel_linf(C[k], Cs[k]) for k in range(N))
        eu = rel_linf(u, us)
        print(wl.shape, "C %.2e u %.2e" % (eC, eu), flush=True)
        assert eC < bar[0] and eu < bar[1]
    b.close()


@pytest.mark.parametrize("dim,shape", [(2, (40, 70)), (3, (8, 9, 20))])
def test_long_calls_on_a_captured_stream(dim, shape):
    """A context that already runs captured groups of its own: while the
    caller captures its stream, ddcc_step records single launches there, and
    each replay is that many steps, between eager calls too. Every state bit
    for bit that of a context without a capture."""
    import torch
    from paper_2311_10314_amd.ddcc import Sim
    wl = W.random_small(dim, 2, shape, seed=63)
    stream = torch.cuda.Stream()
    a = Sim.from_workload(wl, "fp32", stream=stream.cuda_stream)
    b = Sim.from_workload(wl, "fp32")
    for n in (128, 100):
        a.step(n)
        b.step(n)
    a.sync()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        a.step(40)
    print(shape, "captured", flush=True)
    for k in range(4):
        with torch.cuda.stream(stream):
            graph.replay()
        if k:
            a.step(30 * k)
            b.step(30 * k)
        b.step(40)
        a.sync()
        # the capture advanced the context's clock, the replays did not
        x, y = a.save(), b.save()
        assert np.array_equal(x[56:], y[56:]), k
        torch.cuda.synchronize()
    a.close()
    b.close()


@pytest.mark.parametrize("copies", [(5, 6), (14, 15)])
def test_adjoint_of_boxes_that_fill_the_chip(copies):
    """79 200 and 554 400 nodes: fields of six states and of one at a time.
    Every copy of the small box goes through the same arithmetic, so each
    copy's gradient is the small box's over the number of copies, up to the
    order of the two sums in J (relative n 2^-53 < 1e-10 each)."""
    from paper_2311_10314_amd.ddcc import Sim
    small = W.random_small(2, 2, (44, 60), seed=64)
    rep = lambda v: _rep(v, copies)
    big = _repeated(small, copies)
    w = np.random.default_rng(65).uniform(0.0, 1.0, size=(44, 60))
    out = []
    for wl, weight in ((small, w), (big, rep(w))):
        print(wl.shape, flush=True)
        s = Sim.from_workload(wl, "fp64")
        out.append(s.adjoint(7, 3, 0, weight) + (s.time,))
        s.close()
    (J, gc, gp, t), (Jb, gcb, gpb, tb) = out
    m = copies[0] * copies[1]
    assert t == tb == 7
    assert abs(Jb - J) <= 1e-9 * abs(J)
    for g, gb in ((gc, gcb), (gp, gpb)):
        err = np.abs(m * gb - rep(g)).max() / np.abs(g).max()
        print("rel %.2e" % err, flush=True)
        assert err < 1e-9
