"""The second population buffer is the caller's choice: a card without room for it, or
a caller that declines it, gets the same lattice on the smaller aux buffer, with the
same results."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2307_11752_amd import _lib  # noqa: E402
from paper_2307_11752_amd import workloads as W  # noqa: E402

SIZES = {0: 8, 1: 4, 2: 2, 3: 2}


def _pad(b):
    return -(-b // 256) * 256


def _sizes(lib, d, shape, storage):
    p, a, least = (ctypes.c_size_t() for _ in range(3))
    assert lib.lbm_required_bytes(d, *shape, storage, ctypes.byref(p), ctypes.byref(a)) == 0
    assert lib.lbm_min_aux_bytes(d, *shape, storage, ctypes.byref(least)) == 0
    return p.value, a.value, least.value


@pytest.mark.parametrize("storage", sorted(SIZES))
@pytest.mark.parametrize("d,shape", [(1, (5, 4, 3)), (1, (101, 77, 53)), (0, (730, 150, 1)),
                                     (1, (608, 608, 300)), (1, (608, 608, 600))])
def test_smallest_aux_buffer(d, shape, storage):
    """Link words, moving-link words, classes, the result line and 32 bytes a cell of
    scratch between 64 KiB and 1 MiB; the second buffer on top of that below 2^32 bytes."""
    lib = _lib.load()
    pop, aux, least = _sizes(lib, d, shape, storage)
    n = shape[0] * shape[1] * shape[2]
    scratch = min(max(32 * n, 1 << 16), 1 << 20)
    assert least == 2 * _pad(4 * n) + _pad(n) + 256 + _pad(scratch)
    assert aux == least + (pop if pop < 2**32 else 0)


def test_smallest_aux_buffer_of_a_batch():
    lib = _lib.load()
    p, a, least = (ctypes.c_size_t() for _ in range(3))
    shapes = [(62, 9, 4), (65, 7, 5), (33, 21, 40)]
    dims = (ctypes.c_int * 9)(*[v for s in shapes for v in s])
    for storage in SIZES:
        assert lib.lbm_batch_required_bytes(1, 3, dims, storage, ctypes.byref(p), ctypes.byref(a)) == 0
        assert lib.lbm_batch_min_aux_bytes(1, 3, dims, storage, ctypes.byref(least)) == 0
        if SIZES[storage] == 2:  # such batches take no passes
            assert a.value == least.value
        else:
            assert a.value > least.value + p.value
    assert lib.lbm_batch_min_aux_bytes(1, 0, dims, 1, ctypes.byref(least)) == _lib.ERR_ARG
    assert lib.lbm_min_aux_bytes(0, 8, 8, 2, 1, ctypes.byref(least)) == _lib.ERR_ARG


def _lattice(d, shape, **kw):
    import paper_2307_11752_amd as P

    lat = P.Lattice(d, shape, 0.7, **kw)
    lat.set_geometry(W.random_geometry(d, shape, 1, seed=5), 1)
    lat.set_body_force((1e-4, -3e-5, 0.0))
    lat.init_equilibrium(None, W.random_velocity(shape, 3, dim=3 if d else 2))
    return [lat], lat


def _batch(d, shapes, **kw):
    import paper_2307_11752_amd as P

    b = P.Batch(d, shapes, [0.6 + 0.1 * k for k in range(len(shapes))], **kw)
    for m, s in zip(b, shapes):
        m.init_equilibrium(None, W.random_velocity(s, 3, dim=3 if d else 2))
    return list(b), b


MAKE = {"box": lambda **kw: _lattice(1, (40, 24, 12), **kw),
        "plane": lambda **kw: _lattice(0, (130, 51, 1), **kw),
        "batch": lambda **kw: _batch(1, [(40, 24, 12), (16, 9, 7)], **kw)}


@pytest.mark.gpu
@pytest.mark.parametrize("kind", sorted(MAKE))
def test_declined_or_without_room(kind, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no ROCm GPU visible")
    print(f"[second] {kind}", flush=True)
    states, own = MAKE[kind]()
    full = own.aux.numel()
    assert full > own.pop.numel()

    declined = MAKE[kind](second_buffer=False)
    empty = torch.empty

    def no_room(*args, **kw):
        if args and args[0] == full:
            raise torch.OutOfMemoryError("no room")
        return empty(*args, **kw)

    with monkeypatch.context() as m:
        m.setattr(torch, "empty", no_room)
        full_card = MAKE[kind]()
    for other in (declined, full_card):
        assert other[1].aux.numel() < full - own.pop.numel() + 256
    for n in (4, 9, 6):
        for _, o in ((states, own), declined, full_card):
            o.step(n)
        for other in (declined, full_card):
            for a, b in zip(states, other[0]):
                assert torch.equal(a.get_populations(), b.get_populations())
                for x, y in zip(a.moments(), b.moments()):
                    assert np.array_equal(x, y)
