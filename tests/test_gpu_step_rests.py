"""Calls whose length is no multiple of the steps a launch takes: every remainder, on lattices
whose launches take four to eight steps, bitwise against single steps; and the same on contexts
of which a call was captured into a caller's graph, which have to end in the lattice that single
steps end in."""
import numpy as np
import pytest

import synthetic
from gpu_util import announce

pytestmark = pytest.mark.gpu

# squares of four, five, six and four steps (several rounds); strips of eight and six
SIZES = [(150, 50), (340, 330), (285, 283), (611, 590), (1216, 912)]
TILED = [(160, 48), (336, 320), (288, 272), (608, 592), (1216, 912)]


def make(nx, ny, dtype, layout, mrt, solid=0.1):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_13241_amd as lbm
    m = synthetic.random_mask(nx, ny, seed=3, solid_fraction=solid, walls=True)
    lat = lbm.Lattice(m, 0.7, force=(2e-4, -1e-4), dtype=dtype, layout=layout)
    if mrt:
        lat.set_mrt((1.64, 1.54, 1.9))
    lat.init_equilibrium(*synthetic.random_fields(nx, ny, seed=4, u_amp=0.03))
    return lat


def state(lat):
    import torch
    s = torch.zeros(lat.state_bytes(), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()  # the lattice may have a stream of its own
    lat.save_state(s)
    torch.cuda.synchronize()
    return s


def sizes(layout):
    return TILED if layout == "tiled16" else SIZES


@pytest.mark.parametrize("size", range(5))
@pytest.mark.parametrize("layout", ["dense_ab", "dense_aa", "indirect", "tiled16"])
@pytest.mark.parametrize("dtype,mrt", [("f64", False), ("f64", True), ("f32", False)])
def test_every_remainder(dtype, mrt, layout, size):
    import torch
    nx, ny = sizes(layout)[size]
    announce(f"rests {nx}x{ny} {dtype} {layout} mrt={mrt}")
    a, b = make(nx, ny, dtype, layout, mrt), make(nx, ny, dtype, layout, mrt)
    for n in range(1, 19):
        a.step(n)
        for _ in range(n):
            b.step(1)
        assert torch.equal(state(a), state(b)), n
    assert np.isfinite(a.mass())
    a.close()
    b.close()


@pytest.mark.parametrize("layout", ["dense_ab", "dense_aa", "indirect", "tiled16"])
@pytest.mark.parametrize("size", range(5))
def test_captured_contexts_keep_their_lattice(size, layout):
    """step(6) captured, replayed after eager calls of every even length up to 34."""
    import torch
    nx, ny = sizes(layout)[size]
    announce(f"rests of captured contexts {nx}x{ny} {layout}")
    a, b = make(nx, ny, "f32", layout, False), make(nx, ny, "f32", layout, False)
    stream = torch.cuda.Stream()
    a.set_stream(stream)
    a.step(3)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        a.step(6)  # recorded, not run
    b.step(3)
    for n in range(2, 35, 2):
        with torch.cuda.stream(stream):
            graph.replay()
        a.step(n)
        torch.cuda.synchronize()
        for _ in range(6 + n):
            b.step(1)
        assert torch.equal(state(a), state(b)), n
    a.close()
    b.close()
