"""Passes of several steps where they run for long: marches through many planes in
every variant of the kernel, replayed graphs of passes, the full-size lattices of the
benchmark and buffers at the 32-bit offset limit.  All must equal single steps (or
the exact shift of pure streaming) bit for bit; single steps are held to the oracle
elsewhere."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from _pass_cases import MARCHES  # noqa: E402
from paper_2307_11752_amd import workloads as W  # noqa: E402


@pytest.fixture(scope="module")
def lbm():
    if not torch.cuda.is_available():
        pytest.skip("no ROCm GPU visible")
    import paper_2307_11752_amd as P
    from paper_2307_11752_amd import _lib

    _lib.load()
    return P


def _same(a, b):
    x, y = a.get_populations(), b.get_populations()
    assert torch.equal(x, y), int((x != y).sum())


def _pair(lbm, d, shape, storage, walls, **kw):
    """Two lattices in the same state; walls: random, some moving; a body force acts."""
    periodic = 0b001 if walls else (0b111 if d else 0b011)
    nx, ny, nz = shape
    mat = W.random_geometry(d, shape, periodic, seed=5) if walls else np.ones((nz, ny, nx), np.uint8)
    rho, u = W.random_density(shape, 2), W.random_velocity(shape, 3, dim=3 if d else 2)
    out = []
    for _ in range(2):
        lat = lbm.Lattice(d, shape, 0.7, storage=storage, shifted=storage != "f64", **kw)
        lat.set_geometry(mat, periodic)
        lat.set_body_force((1e-4, -3e-5, 0.0))
        lat.set_wall_velocity((0.03, 0.0, 0.0))
        lat.init_equilibrium(rho, u)
        out.append(lat)
    return out


def _single(lat, n):
    for _ in range(n):
        lat.step(1)


@pytest.mark.parametrize("shape,storage,walls", [m[:3] for m in MARCHES])
def test_long_marches(lbm, shape, storage, walls):
    print(f"[march] {shape} {storage} walls={walls}", flush=True)
    run, one = _pair(lbm, 1, shape, storage, walls)
    for n in (4, 3, 9, 8, 6):
        run.step(n)
        _single(one, n)
        _same(run, one)


# Graphs long enough that runs are replayed: eight passes or more (16 steps of D3Q19,
# 128 of D2Q9 whatever its passes hold).  Walled 16-bit lattices of 65536 and more
# cells round by the parity of the step.
@pytest.mark.parametrize("d,shape,storage,walls,length", [
    (1, (40, 24, 20), "f32", False, 16), (1, (40, 24, 20), "f64", True, 18),
    (1, (96, 48, 32), "f16", True, 18), (1, (96, 48, 32), "bf16", True, 20),
    (1, (90, 60, 30), "f16", False, 22), (0, (512, 300, 1), "f16", True, 130),
    (0, (130, 51, 1), "f32", True, 128), (0, (64, 64, 1), "f64", False, 134)])
def test_replays_of_passes(lbm, d, shape, storage, walls, length):
    print(f"[replay] {shape} {storage} walls={walls} {length}", flush=True)
    run, one = _pair(lbm, d, shape, storage, walls, stream=torch.cuda.Stream())
    run.set_graph_steps(length)
    for n in (length, 1, length, 2 * length + 5, 3, length + 2, 1, 2 * length):
        run.step(n)
        _single(one, n)
        run.moments_device()  # eager work between replays
        _same(run, one)
    run.set_tau(0.9)
    one.set_tau(0.9)
    run.step(length)
    _single(one, length)
    _same(run, one)


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("d,shapes", [(1, [(62, 9, 4), (33, 21, 40), (16, 16, 16)]),
                                      (0, [(254, 4, 1), (257, 37, 1), (61, 64, 1)])])
def test_replays_of_batch_passes(lbm, d, shapes, storage):
    print(f"[replay] batch {shapes} {storage}", flush=True)
    runs = [lbm.Batch(d, shapes, [0.6, 0.7, 0.8], storage=storage, shifted=storage != "f64")
            for _ in range(2)]
    for b in runs:
        assert b.aux.numel() > b.pop.numel()  # the second buffer is there: passes are taken
        for k, (m, s) in enumerate(zip(b, shapes)):
            m.init_equilibrium(W.random_density(s, k), W.random_velocity(s, k, dim=3 if d else 2))
    run, one = runs
    for length in (16, 18):
        run.set_graph_steps(length)
        for n in (length, 1, length, 2 * length + 5, 3, length + 2, 1, 2 * length):
            run.step(n)
            _single(one, n)
            for a, b in zip(run, one):
                _same(a, b)
    for b in runs:
        b.close()


@pytest.mark.parametrize("case,storage", [("tgv", "f32"), ("tgv", "f16"), ("channel", "f32"),
                                          ("channel", "f64")])
def test_full_size(lbm, case, storage):
    """Taylor-Green 256^3 and the channel of spheres 512 x 128 x 128."""
    print(f"[full] {case} {storage}", flush=True)
    wl = W.tgv3d(256, u0=0.05, tau=0.8) if case == "tgv" else W.channel_spheres()
    u = wl.u0 if wl.u0 is not None else W.random_velocity(wl.shape, 11, amplitude=0.02)
    lats = []
    for _ in range(2):
        lat = lbm.Lattice(1, wl.shape, wl.tau, storage=storage, shifted=storage != "f64")
        lat.set_geometry(wl.material, wl.periodic)
        lat.set_body_force(wl.g)
        lat.init_equilibrium(None, u)
        lats.append(lat)
    run, one = lats
    for n in (4, 5, 4):
        run.step(n)
        _single(one, n)
        _same(run, one)


@pytest.mark.parametrize("shape,storage", [((380, 380, 380), "f32"), ((480, 480, 480), "f16")])
def test_streaming_at_the_offset_limit(orc, lbm, shape, storage):
    """Pure streaming (omega = 0) moves every population by n c_i: buffers just under
    2^32 bytes, through passes that end in either form."""
    nx, ny, nz = shape
    print(f"[limit] {shape} {storage}", flush=True)
    c, w, _, _ = orc.descriptor(1)
    lat = lbm.Lattice(1, shape, float("inf"), storage=storage, shifted=True)
    assert 0.97 * 2**32 < lat.pop.numel() < 2**32 and lat.aux.numel() > lat.pop.numel()
    lat.set_geometry(np.ones((nz, ny, nx), np.uint8), 7)
    dev = torch.device("cuda")
    z = torch.arange(nz, device=dev, dtype=torch.int64).view(nz, 1, 1)
    y = torch.arange(ny, device=dev, dtype=torch.int64).view(1, ny, 1)
    x = torch.arange(nx, device=dev, dtype=torch.int64).view(1, 1, nx)

    def initial(i):
        m = (7 * x + 13 * y + 29 * z + 5 * i) % 64 - 32
        return w[i] + m.to(torch.float64) * 2.0**-16

    f = torch.empty((19, nz, ny, nx), dtype=torch.float64, device=dev)
    for i in range(19):
        f[i] = initial(i)
    lat.set_populations(f)
    del f
    done = 0
    for n in (4, 5, 4):  # natural to natural, one step then passes, swapped to swapped
        lat.step(n)
        done += n
        print(f"[limit] {shape} {storage}: after {done} steps", flush=True)
        got = lat.get_populations()
        for i in range(19):
            shift = tuple(done * int(c[i][a]) for a in (2, 1, 0))
            assert torch.equal(got[i], torch.roll(initial(i), shifts=shift, dims=(0, 1, 2))), (done, i)
        del got
    lat.close()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("d,shape,storage", [(1, (64, 48, 40), "f32"), (1, (61, 47, 35), "f64"),
                                             (0, (700, 301, 1), "f16"), (0, (700, 301, 1), "f64")])
def test_fields_in_one_copy_and_in_chunks(lbm, d, shape, storage):
    """lbm_moments through the second population buffer (D2Q9 in 16 bits: two chunks) and
    through the scratch (32768 cells a chunk), in both propagation phases."""
    print(f"[fields] {shape} {storage}", flush=True)
    wide, _ = _pair(lbm, d, shape, storage, True)
    chunks, _ = _pair(lbm, d, shape, storage, True, second_buffer=False)
    for n in (2, 3):
        wide.step(n)
        chunks.step(n)
        _same(wide, chunks)
        (r1, u1), (r2, u2) = wide.moments(), chunks.moments()
        assert np.array_equal(r1, r2) and np.array_equal(u1, u2)
