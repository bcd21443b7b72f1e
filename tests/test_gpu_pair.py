"""Runs of four and more steps advance two steps per pass between two population
buffers.  The same cell arithmetic runs in every kernel, so such a run must equal
its steps taken one by one, and the run of a lattice created without the second
buffer, bit for bit.  Shapes at the edges of the passes' tiles: rows of one, two
and three waves more or less one cell, the shortest march that takes passes (4
planes) and one that does not, one plane per work-group, odd edges, walls (some
moving) on and off the tile borders."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lbm():
    if not torch.cuda.is_available():
        pytest.skip("no ROCm GPU visible")
    import paper_2307_11752_amd as P
    from paper_2307_11752_amd import _lib

    _lib.load()
    return P


from paper_2307_11752_amd import workloads as W  # noqa: E402

SHAPES = [(1, (62, 9, 4)), (1, (65, 7, 5)), (1, (64, 16, 3)), (1, (130, 6, 9)), (1, (19, 21, 40)),
          (1, (96, 33, 12)), (1, (7, 5, 4)), (0, (254, 4, 1)), (0, (257, 37, 1)), (0, (61, 64, 1)),
          (0, (12, 3, 1))]


def _lattice(lbm, d, shape, storage, walls, second=True):
    periodic = 0b001 if walls else (0b111 if d else 0b011)
    nx, ny, nz = shape
    mat = W.random_geometry(d, shape, periodic, seed=5) if walls else np.ones((nz, ny, nx), np.uint8)
    lat = lbm.Lattice(d, shape, 0.7, storage=storage, shifted=storage != "f64")
    if not second:  # recreate the handle on an aux buffer without the second population buffer
        lib = lat.lib
        lib.lbm_lattice_destroy(lat.h)
        cells = nx * ny * nz
        scratch = min(max(32 * cells, 1 << 16), 1 << 20)
        pad = lambda b: -(-b // 256) * 256  # noqa: E731
        aux = 2 * pad(4 * cells) + pad(cells) + 256 + pad(scratch)
        h = ctypes.c_void_p()
        assert lib.lbm_lattice_create(ctypes.byref(h), d, nx, ny, nz, 0.7,
                                      {"f64": 0, "f32": 1, "f16": 2, "bf16": 3}[storage],
                                      1 if storage != "f64" else 0,
                                      ctypes.c_void_p(lat.pop.data_ptr()), lat.pop.numel(),
                                      ctypes.c_void_p(lat.aux.data_ptr()), aux,
                                      ctypes.c_void_p(lat.stream.cuda_stream)) == 0
        lat.h = h
    lat.set_geometry(mat, periodic)
    lat.set_body_force((1e-4, -3e-5, 0.0))
    lat.set_wall_velocity((0.03, 0.0, 0.0))
    lat.init_equilibrium(W.random_density(shape, 2),
                         W.random_velocity(shape, 3, dim=3 if d else 2))
    return lat


@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("d,shape", SHAPES)
def test_passes_equal_single_steps(lbm, d, shape, storage, walls):
    print(f"[pair] d={d} {shape} {storage} walls={walls}", flush=True)
    run = _lattice(lbm, d, shape, storage, walls)
    one = _lattice(lbm, d, shape, storage, walls)
    alone = _lattice(lbm, d, shape, storage, walls, second=False)
    for n in (4, 3, 9, 6):  # from both propagation phases, with every remainder
        run.step(n)
        alone.step(n)
        for _ in range(n):
            one.step(1)
        a, b, c = run.get_populations(), one.get_populations(), alone.get_populations()
        assert torch.equal(a, b), int((a != b).sum())
        assert torch.equal(c, b), int((c != b).sum())
    assert run.info()[0] == 22


def test_too_small_aux_is_refused(lbm):
    lat = lbm.Lattice(1, (16, 16, 16), 0.7)
    cells, pad = 4096, 256
    least = 9 * cells + pad + 32 * cells
    h = ctypes.c_void_p()
    args = (1, 16, 16, 16, 0.7, 1, 0, ctypes.c_void_p(lat.pop.data_ptr()), lat.pop.numel(),
            ctypes.c_void_p(lat.aux.data_ptr()))
    assert lat.lib.lbm_lattice_create(ctypes.byref(h), *args, least - 256, None) == -1
    assert lat.lib.lbm_lattice_create(ctypes.byref(h), *args, least, None) == 0
    assert lat.lib.lbm_lattice_destroy(h) == 0


BATCHES = {
    "boxes": (1, [(62, 9, 4), (65, 7, 5), (16, 16, 16), (33, 21, 40), (7, 5, 4), (130, 6, 9)]),
    "cut": (1, [(48, 40, 44)] * 3 + [(9, 8, 11)] * 17),  # members cut over the XCDs and whole ones
    "planes": (0, [(254, 4, 1), (257, 37, 1), (61, 64, 1), (12, 5, 1)]),
    "short": (1, [(20, 12, 10), (9, 9, 3)]),  # a march too short: the batch steps in place
}


@pytest.mark.parametrize("graph", [0, 6])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("name", BATCHES)
def test_batch_passes_equal_single_steps(lbm, name, storage, graph):
    print(f"[pair] batch {name} {storage} graph={graph}", flush=True)
    d, shapes = BATCHES[name]
    taus = [0.55 + 0.4 * k / len(shapes) for k in range(len(shapes))]
    runs = [lbm.Batch(d, shapes, taus, storage=storage, shifted=storage != "f64") for _ in range(2)]
    runs[0].set_graph_steps(graph)
    for b in runs:
        for k, (m, s) in enumerate(zip(b, shapes)):
            m.init_equilibrium(W.random_density(s, k), W.random_velocity(s, k, dim=3 if d else 2))
    for n in (4, 3, 9, 6, 13):
        runs[0].step(n)
        for _ in range(n):
            runs[1].step(1)
        for a, b in zip(*runs):
            x, y = a.get_populations(), b.get_populations()
            assert torch.equal(x, y), (a.index, int((x != y).sum()))
    assert runs[0][0].info()[0] == 35
    for b in runs:
        b.close()


# Regions of 256 to 4096 cells, narrower and wider than the lattice, passes of
# different lengths in one run; the walled 512 x 300 takes the flat in-place kernel.
DEEP_SHAPES = [(5, 4, 1), (17, 9, 1), (64, 64, 1), (130, 51, 1), (333, 201, 1), (512, 300, 1),
               (1023, 511, 1)]


@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("shape", DEEP_SHAPES)
def test_deep_passes_equal_single_steps(lbm, shape, storage, walls):
    print(f"[deep] {shape} {storage} walls={walls}", flush=True)
    run = _lattice(lbm, 0, shape, storage, walls)
    one = _lattice(lbm, 0, shape, storage, walls)
    for n in (4, 1, 31, 5, 18):
        run.step(n)
        for _ in range(n):
            one.step(1)
        a, b = run.get_populations(), one.get_populations()
        assert torch.equal(a, b), int((a != b).sum())
    assert run.info()[0] == 59


# A caller's own graph of an even number of steps returns to the phase it was
# captured in, and can be replayed any number of times.
@pytest.mark.parametrize("kind", ["box", "walls", "plane", "batch"])
def test_captured_steps_replay(lbm, kind):
    print(f"[pair] captured {kind}", flush=True)
    shape = (40, 24, 1) if kind == "plane" else (40, 24, 12)
    d, walls = int(kind != "plane"), kind in ("walls", "plane")
    stream = torch.cuda.Stream()

    def make():
        if kind == "batch":
            b = lbm.Batch(1, [shape, (16, 9, 7)], [0.7, 0.8], stream=stream)
            for m, s in zip(b, [shape, (16, 9, 7)]):
                m.init_equilibrium(None, W.random_velocity(s, 3, dim=3))
            return b, list(b)
        lat = lbm.Lattice(d, shape, 0.7, stream=stream)
        lat.set_geometry(W.random_geometry(d, shape, 1, seed=5) if walls
                         else np.ones(shape[::-1], np.uint8), 0b001 if walls else 0b111)
        lat.init_equilibrium(None, W.random_velocity(shape, 3, dim=3 if d else 2))
        return lat, [lat]

    (run, states), (eager, expect) = make(), make()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        run.step(6)
    for _ in range(3):
        with torch.cuda.stream(stream):
            graph.replay()
        torch.cuda.synchronize()
        eager.step(6)
        for a, b in zip(states, expect):
            assert torch.equal(a.get_populations(), b.get_populations())
