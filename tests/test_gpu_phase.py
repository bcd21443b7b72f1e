"""A run of an even number of steps leaves the propagation phase as it was, through
passes of several steps as step by step.  What rests on it: a graph that the
caller captured may be replayed between eager runs and after a new start, and one
member of a batch may be started anew while the others go on.  Every state must
equal, bit for bit, that of single steps."""
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

# Boxes and channels of D3Q19 (passes of two steps: fours of them) and planes of
# D2Q9 (an even number of longer passes); members of a batch all take passes.
KINDS = ["box", "walls", "plane", "cavity", "batch", "flat batch"]
BATCHES = {"batch": (1, [(40, 24, 12), (16, 9, 7)]), "flat batch": (0, [(130, 40, 1), (61, 17, 1)])}


class Case:
    """A lattice or a batch on a stream of its own."""

    def __init__(self, lbm, kind, stream, storage="f32"):
        self.kind, self.stream = kind, stream
        shifted = storage != "f64"
        if kind in BATCHES:
            self.d, self.shapes = BATCHES[kind]
            self.own = lbm.Batch(self.d, self.shapes, [0.7, 0.8], storage=storage, shifted=shifted,
                                 stream=stream)
            self.states = list(self.own)
        else:
            self.d = int(kind in ("box", "walls"))
            self.shapes = [(40, 24, 12) if self.d else (130, 61, 1)]
            self.own = lbm.Lattice(self.d, self.shapes[0], 0.7, storage=storage, shifted=shifted,
                                   stream=stream)
            nx, ny, nz = self.shapes[0]
            periodic = {"box": 0b111, "plane": 0b011, "walls": 0b001, "cavity": 0}[kind]
            mat = np.ones((nz, ny, nx), np.uint8) if kind in ("box", "plane") else \
                W.random_geometry(self.d, self.shapes[0], periodic, seed=5)
            self.own.set_geometry(mat, periodic)
            self.own.set_body_force((1e-4, -3e-5, 0.0))
            self.own.set_wall_velocity((0.03, 0.0, 0.0))
            self.states = [self.own]
        self.start(3)

    def start(self, seed):
        for m, s in zip(self.states, self.shapes):
            m.init_equilibrium(W.random_density(s, seed + 1),
                               W.random_velocity(s, seed, dim=3 if self.d else 2))

    def single(self, n):
        for _ in range(n):
            self.own.step(1)

    def capture(self, n):
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=self.stream):
            self.own.step(n)
        return graph

    def replay(self, graph):
        with torch.cuda.stream(self.stream):
            graph.replay()
        torch.cuda.synchronize()


def _same(a, b):
    for x, y in zip(a.states, b.states):
        p, q = x.get_populations(), y.get_populations()
        assert torch.equal(p, q), int((p != q).sum())


@pytest.mark.parametrize("n", [2, 6, 8])
@pytest.mark.parametrize("kind", KINDS)
def test_replays_between_eager_runs(lbm, kind, n):
    """Captured in either phase, replayed after eager runs of even lengths."""
    print(f"[phase] {kind} captured {n}", flush=True)
    stream = torch.cuda.Stream()
    run, one = Case(lbm, kind, stream), Case(lbm, kind, stream)
    for before in (0, 3):
        run.own.step(before)
        one.single(before)
        graph = run.capture(n)  # records the steps, none is taken yet
        for eager in (0, 4, 10, 16):
            run.own.step(eager)
            one.single(eager)
            run.replay(graph)
            one.single(n)
            _same(run, one)
        run.start(7 + before)
        one.start(7 + before)


@pytest.mark.parametrize("kind", KINDS)
def test_replays_after_a_warm_up_and_a_new_start(lbm, kind):
    print(f"[phase] {kind} warm-up", flush=True)
    stream = torch.cuda.Stream()
    run, one = Case(lbm, kind, stream), Case(lbm, kind, stream)
    run.own.step(4)  # warm-up
    graph = run.capture(6)
    for seed in (11, 12):
        run.start(seed)
        one.start(seed)
        for _ in range(3):
            run.replay(graph)
            one.single(6)
            _same(run, one)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("kind", sorted(BATCHES))
def test_a_member_started_anew(lbm, kind, storage):
    """After an even number of steps one member may be given new populations; after
    an odd one the members' phases differ and the step is refused, as ever."""
    print(f"[phase] {kind} {storage}: a member started anew", flush=True)
    from paper_2307_11752_amd import _lib

    stream = torch.cuda.Stream()
    run, one = (Case(lbm, kind, stream, storage) for _ in range(2))
    shape = run.shapes[1]
    u = W.random_velocity(shape, 21, dim=3 if run.d else 2)
    for n in (4, 6, 20):
        run.own.step(n)
        one.single(n)
        for c in (run, one):
            c.states[1].init_equilibrium(None, u)
        run.own.step(8)
        one.single(8)
        _same(run, one)
    run.own.step(5)
    run.states[1].init_equilibrium(None, u)
    with pytest.raises(_lib.LBMError) as e:
        run.own.step(4)
    assert e.value.status == _lib.ERR_STATE


@pytest.mark.parametrize("storage", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("kind", KINDS)
def test_runs_of_every_remainder(lbm, kind, storage):
    """Runs of 4 to 11 steps from both phases: passes that begin and end in either form."""
    print(f"[phase] {kind} {storage}: remainders", flush=True)
    stream = torch.cuda.Stream()
    run, one = (Case(lbm, kind, stream, storage) for _ in range(2))
    for n in (4, 8, 6, 5, 4, 8, 7, 9, 10, 11, 4):
        run.own.step(n)
        one.single(n)
        _same(run, one)
