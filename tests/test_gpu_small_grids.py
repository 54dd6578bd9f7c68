"""Launch shapes and step modes that the grid size chooses, against the oracle.

2D boxes whose tiles fit the compute units run in wide workgroups (a thread
per halo node): one-tile boxes, partial tiles in x and y, and the largest
boxes of the 64 x 2 and 64 x 4 shapes. 3D boxes take shorter z columns: one
plane per workgroup, a last column with fewer planes than the others, one
tile; boxes at most 32 nodes wide 32 x 8 tiles. Bars: the method's own, FP64
1e-10 and FP32 1e-5 on C_i and u; FP16 storage (three phases: the plane
pipeline) as in test_gpu_halfstore, C 10 u_s and u 50 u_s with u_s = 2^-11.
"""
import numpy as np
import pytest

from paper_2311_10314_amd import workloads as W
from tests.helpers import oracle_run, rel_linf

pytestmark = pytest.mark.gpu

BAR = {"fp64": (1e-10, 1e-10), "fp32": (1e-5, 1e-5),
       "fp16": (10 * 2.0 ** -11, 50 * 2.0 ** -11)}


def _check(wl, precision, steps, tile=0):
    from paper_2311_10314_amd.ddcc import Sim
    print(wl.shape, wl.nphase, precision, "tile", tile, flush=True)
    sim = Sim.from_workload(wl, precision)
    sim.set_tile(0, tile)
    sim.step(steps)
    C, u, _ = sim.read_moments()
    sim.close()
    o = oracle_run(wl, steps)
    eC = max(rel_linf(C[i], o["C"][i]) for i in range(wl.nphase))
    eu = rel_linf(u, o["u"])
    print("C %.2e u %.2e" % (eC, eu), flush=True)
    assert eC < BAR[precision][0] and eu < BAR[precision][1]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("N,shape", [(2, (1, 64)), (3, (3, 65)), (4, (5, 130)),
                                     (2, (128, 128)), (3, (127, 127)),
                                     (2, (256, 200)), (3, (253, 255))])
def test_wide_workgroups(N, shape, precision):
    _check(W.random_small(2, N, shape, seed=41), precision, 4)


@pytest.mark.parametrize("tile", [2, 4])
def test_wide_workgroups_by_tile(tile):
    """Both heights of the wide shape on one box (64 x 4: float only)."""
    _check(W.random_small(2, 2, (129, 129), seed=42), "fp32", 4, tile)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("N,lattice,shape", [(2, "D3Q15", (5, 3, 20)),
                                             (2, "D3Q15", (17, 30, 66)),
                                             (3, "D3Q7", (7, 50, 100)),
                                             (2, "D3Q15", (9, 17, 32)),
                                             (3, "D3Q15", (10, 15, 33))])
def test_short_columns(N, lattice, shape, precision):
    prm = {"d0": 0.3} if lattice == "D3Q7" else {}
    _check(W.random_small(3, N, shape, seed=43, lattice_f=lattice, **prm),
           precision, 3)


@pytest.mark.parametrize("N,lattice,shape", [(2, "D3Q15", (9, 10, 65)),
                                             (3, "D3Q7", (11, 17, 96)),
                                             (2, "D3Q7", (6, 13, 129)),
                                             (3, "D3Q15", (5, 8, 160))])
def test_float64_rows_in_32_node_tiles(N, lattice, shape):
    """Boxes several 32 x 8 tiles wide, the last one partly filled or full."""
    prm = {"d0": 0.3} if lattice == "D3Q7" else {}
    _check(W.random_small(3, N, shape, seed=48, lattice_f=lattice, **prm),
           "fp64", 3)


@pytest.mark.parametrize("lattice", ["D3Q15", "D3Q7"])
def test_half_storage_three_phases(lattice):
    prm = {"d0": 0.3} if lattice == "D3Q7" else {}
    _check(W.random_small(3, 3, (11, 22, 70), seed=44, lattice_f=lattice,
                          **prm), "fp16", 3)


@pytest.mark.parametrize("dim,shape,precision", [(2, (40, 70), "fp32"),
                                                 (2, (33, 64), "fp64"),
                                                 (3, (8, 9, 20), "fp32")])
def test_captured_steps_equal_single_steps(dim, shape, precision):
    """Small boxes launch long calls as captured groups of steps: several
    calls, even and odd, with read-outs, masses and a tile change between
    them, against a context that is stepped one by one, bit for bit."""
    from paper_2311_10314_amd.ddcc import Sim
    wl = W.random_small(dim, 2, shape, seed=45)
    a = Sim.from_workload(wl, precision)
    b = Sim.from_workload(wl, precision)
    for k, n in enumerate([128, 150, 201, 90, 300]):
        if k == 3:
            a.set_tile(0, 4)
            b.set_tile(0, 4)
        a.step(n)
        for _ in range(n):
            b.step(1)
        x, y = a.read_moments(), b.read_moments()
        print(shape, "after", a.time, flush=True)
        assert a.time == b.time
        assert all(np.array_equal(p, q) for p, q in zip(x, y))
        assert np.array_equal(a.mass(), b.mass())
        assert np.array_equal(a.save(), b.save())
    a.close()
    b.close()


@pytest.mark.parametrize("N,shape,precision", [(2, (830, 1001), "fp64"),
                                               (3, (811, 801), "fp32"),
                                               (4, (701, 699), "fp16")])
def test_streaming_rows_off_cache_lines(N, shape, precision):
    """2D boxes larger than the memory-side cache whose rows start anywhere:
    streaming load order without nontemporal accesses, partial tiles."""
    _check(W.random_small(2, N, shape, seed=46), precision, 2)


@pytest.mark.parametrize("N,lattice,shape,precision",
                         [(2, "D3Q15", (5, 3, 20), "fp64"),
                          (3, "D3Q7", (7, 9, 33), "fp32"),
                          (3, "D3Q15", (6, 5, 63), "fp16"),
                          (2, "D3Q15", (3, 70, 97), "bf16"),
                          (2, "D3Q15", (4, 6, 64), "fp32"),
                          (3, "D3Q7", (6, 5, 70), "fp64"),
                          (2, "D3Q15", (5, 9, 100), "fp32"),
                          (3, "D3Q15", (4, 7, 127), "fp16"),
                          (2, "D3Q15", (3, 10, 130), "bf16")])
def test_rows_of_any_length_3d(N, lattice, shape, precision):
    """Planes whose rows are padded on the device: a state moved between two
    contexts through its dense checkpoint goes on bit for bit, and the mass is
    the sum of the checkpoint's populations (float64 additions in another
    order: each term is rounded once per addition at most)."""
    from paper_2311_10314_amd.ddcc import Sim
    prm = {"d0": 0.3} if lattice == "D3Q7" else {}
    wl = W.random_small(3, N, shape, seed=47, lattice_f=lattice, **prm)
    a, b = Sim.from_workload(wl, precision), Sim.from_workload(wl, precision)
    a.step(3)
    state = a.save()
    b.load(state)
    assert np.array_equal(b.save(), state)
    for _ in range(2):
        a.step(1)
        b.step(1)
        assert np.array_equal(a.save(), b.save())
    assert all(np.array_equal(x, y)
               for x, y in zip(a.read_moments(), b.read_moments()))
    n, q = int(np.prod(shape)), 15 if lattice == "D3Q15" else 7
    raw = a.save()[56:]
    esz = {"fp64": 8, "fp32": 4}.get(precision, 2)
    f = raw[:N * (q - 1) * n * esz].copy()
    f = ((f.view(np.uint16).astype(np.uint32) << 16).view(np.float32)
         if precision == "bf16" else f.view("f%d" % esz))
    f0 = raw[f.size * esz:][:N * n * 8].copy().view(np.float64)
    f = np.concatenate([f0.reshape(N, n),
                        f.astype(np.float64).reshape(N, -1)], axis=1)
    tol = 2 * n * q * 2.0 ** -53 * np.abs(f).sum(axis=1)
    assert np.all(np.abs(a.mass() - f.sum(axis=1)) <= tol)
    a.close()
    b.close()
