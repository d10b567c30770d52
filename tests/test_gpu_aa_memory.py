"""The AA layout holds one lattice: steps of several per launch borrow a second one for the
length of a call, from memory that the caller lends, and give it back.

Memory held after a call; raw states against single in-place steps with the lent memory full of
NaN patterns (nothing of it may reach the state), for call lengths that leave every remainder;
memory that is too small, absent, refused or not to be used."""
import ctypes

import numpy as np
import pytest

import synthetic
from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lbm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_13241_amd as m
    m.load()
    return m


def make(lbm, shape, dtype, solid=True):
    if len(shape) == 2:
        nx, ny = shape
        m = (synthetic.random_mask(nx, ny, seed=5, solid_fraction=0.1, walls=True) if solid
             else synthetic.all_fluid(nx, ny))
        lat = lbm.Lattice(m, 0.7, force=(2e-4, -1e-4), dtype=dtype, layout="dense_aa")
        lat.init_equilibrium(*synthetic.random_fields(nx, ny, seed=6, u_amp=0.03))
        return lat
    nx, ny, nz = shape
    m = (synthetic.random_mask3(nx, ny, nz, seed=7, solid_fraction=0.1, walls=True) if solid
         else np.zeros((nz, ny, nx), np.uint8))
    lat = lbm.Lattice3D(m, 0.7, dtype=dtype, layout="dense_aa")
    lat.init_equilibrium(*synthetic.random_fields3(nx, ny, nz, seed=8))
    return lat


def state(lat):
    import torch
    s = torch.zeros(lat.state_bytes(), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()  # the lattice may have a stream of its own
    lat.save_state(s)
    torch.cuda.synchronize()
    return s


def entry(lat, name):
    return getattr(lat._lib, f"lbm{'3d' if hasattr(lat, 'nz') else ''}_{name}")


def wanted(lat, n):
    b = ctypes.c_size_t(1)
    lat._check(entry(lat, "step_scratch_bytes")(lat._ctx, n, ctypes.byref(b)))
    return b.value


SHAPES = [(150, 50), (611, 590), (1216, 912), (65, 66, 128)]


@pytest.mark.parametrize("shape", SHAPES)
def test_memory_is_given_back(lbm, shape):
    import torch
    announce(f"AA memory {shape}")
    lat = make(lbm, shape, "f32")
    blocks, held = set(lbm._torch_blocks), lat.info()["device_bytes"]
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    lat.step(20)
    assert lat.info()["device_bytes"] == held
    assert set(lbm._torch_blocks) == blocks
    assert torch.cuda.memory_allocated() == before
    lat.close()


@pytest.mark.parametrize("shape,dtype", [((150, 50), "f64"), ((150, 50), "f16s"),
                                         ((250, 241), "f32"), ((285, 283), "f64"),
                                         ((611, 590), "f32"), ((1216, 912), "f64"),
                                         ((1216, 912), "f32"), ((65, 66, 128), "f32"),
                                         ((33, 40, 210), "f64")])
@pytest.mark.parametrize("solid", [True, False])
def test_lent_memory_is_only_scratch(lbm, shape, dtype, solid):
    import torch
    announce(f"AA lent memory {shape} {dtype} {solid}")
    a, b = make(lbm, shape, dtype, solid), make(lbm, shape, dtype, solid)
    b.in_place = True
    used = 0
    for n in list(range(1, 14)) + [20, 33]:
        need = wanted(a, n)
        used += need > 0
        block = torch.full((max(need, 1),), 0xFF, dtype=torch.uint8, device="cuda")
        a._check(entry(a, "step_scratch")(a._ctx, n, block.data_ptr(), need))
        b.step(n)
        assert torch.equal(state(a), state(b)), n
    assert used
    assert np.isfinite(a.mass())
    a.close()
    b.close()


@pytest.mark.parametrize("shape", [(150, 50), (65, 66, 128)])
def test_without_memory(lbm, shape, monkeypatch):
    """Too little, none, switched off, a full device, an allocation that fails: refused (too
    little) or in place."""
    import torch
    announce(f"AA without memory {shape}")
    a, b = make(lbm, shape, "f32"), make(lbm, shape, "f32")
    need = wanted(a, 20)
    assert need == a.state_bytes()
    block = torch.empty(need, dtype=torch.uint8, device="cuda")
    assert entry(a, "step_scratch")(a._ctx, 20, block.data_ptr(), need - 1) == -1
    assert a.info()["time_step"] == 0
    a._check(entry(a, "step_scratch")(a._ctx, 20, None, 0))
    a._check(entry(a, "step")(a._ctx, 20))
    assert wanted(a, 1) == wanted(a, 0) == wanted(a, -1) == 0
    assert lbm._spare(1 << 30) and not lbm._spare(5 << 30)
    monkeypatch.setattr(torch.cuda, "mem_get_info", lambda *_: (10 << 30, 288 << 30))
    assert not lbm._spare(1 << 30)
    # blocks that torch holds without using them are free memory
    monkeypatch.setattr(torch.cuda, "memory_stats_as_nested_dict", lambda *_: {
        "reserved_bytes": {"all": {"current": 200 << 30}},
        "allocated_bytes": {"all": {"current": 20 << 30}}})
    assert lbm._spare(1 << 30)
    monkeypatch.setattr(lbm, "_spare", lambda _: False)
    a.step(20)
    monkeypatch.undo()

    def fails(*_, **__):
        raise torch.cuda.OutOfMemoryError("none left")
    monkeypatch.setattr(torch, "empty", fails)
    a.step(20)
    monkeypatch.undo()
    b.in_place = True
    b.step(80)
    assert torch.equal(state(a), state(b))
    dense = lbm.Lattice(synthetic.all_fluid(150, 50), 0.7, layout="dense_ab")
    assert wanted(dense, 20) == 0
    for lat in (a, b, dense):
        lat.close()


@pytest.mark.parametrize("shape", [(150, 50), (65, 66, 128)])
def test_captured_calls_borrow_nothing(lbm, shape):
    import torch
    announce(f"AA captured {shape}")
    a, b = make(lbm, shape, "f32"), make(lbm, shape, "f32")
    stream = torch.cuda.Stream()
    a.set_stream(stream)
    a.step(9)
    block = torch.empty(wanted(a, 8), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        size = wanted(a, 8)
        a._check(entry(a, "step_scratch")(a._ctx, 8, block.data_ptr(), block.numel()))
    assert size == 0
    total = 9
    for eager in (8, 14, 6):
        block.fill_(0xFF)
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            graph.replay()
        a.step(eager)
        torch.cuda.synchronize()
        total += 8 + eager
    b.in_place = True
    b.step(total)
    assert np.array_equal(a.get_populations(), b.get_populations())
    a.close()
    b.close()


def test_steps_beside_a_capture(lbm, monkeypatch):
    """Steps of a lattice on its own stream while another stream is being captured: run, not
    recorded, and without asking for memory."""
    import torch
    announce("AA steps beside a capture")
    a, b = make(lbm, (611, 590), "f32"), make(lbm, (611, 590), "f32")
    own, other = torch.cuda.Stream(), torch.cuda.Stream()
    a.set_stream(own)
    x = torch.zeros(1000, device="cuda")
    torch.cuda.synchronize()
    asked = []
    real = torch.empty
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=other):
        x += 1
        monkeypatch.setattr(torch, "empty", lambda *p, **k: asked.append(p) or real(*p, **k))
        a.step(20)
        monkeypatch.undo()
    graph.replay()
    torch.cuda.synchronize()
    assert not asked and float(x.sum()) == 1000.0
    b.in_place = True
    b.step(20)
    assert torch.equal(state(a), state(b))
    a.close()
    b.close()


def test_threads_and_streams(lbm):
    """Lattices stepped by threads of their own, on streams of their own: each borrows for itself."""
    import threading

    import torch
    announce("AA lattices in four threads")
    shapes = [(150, 50), (611, 590), (1216, 912), (65, 66, 128)]
    lats = [make(lbm, s, "f32") for s in shapes]
    want = [make(lbm, s, "f32") for s in shapes]
    streams = [torch.cuda.Stream() for _ in shapes]
    for lat, stream in zip(lats, streams):
        lat.set_stream(stream)
    torch.cuda.synchronize()
    counts = [9, 20, 5, 16, 33, 8] * 3

    def work(lat):
        for n in counts:
            lat.step(n)

    threads = [threading.Thread(target=work, args=(lat,)) for lat in lats]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for lat, ref in zip(lats, want):
        ref.in_place = True
        ref.step(sum(counts))
        assert torch.equal(state(lat), state(ref))
        lat.close()
        ref.close()
