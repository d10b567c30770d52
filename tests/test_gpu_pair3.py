"""Two D3Q19 steps in one launch against single steps, bitwise: a step(n) call takes pairs,
n step(1) calls take none, and the arithmetic of a node is the same.  The shapes have as few
nodes as pairs are taken for, with one node or a remainder along each axis and around the
columns a workgroup writes (32 or 64 by 13); walls, solids, a body force, the collision models,
every storage type; the A-B layout and the AA layout (pairs start after an odd number of
steps); a state saved between pairs; a step captured by the caller."""
import numpy as np
import pytest

import synthetic
from gpu_util import announce

pytestmark = pytest.mark.gpu

MRT = (1.19, 1.4, 1.64, 1.3, 1.55)


@pytest.fixture(scope="module")
def lbm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_13241_amd as m
    m.load()
    return m


def make(lbm, shape, dtype, layout, solid=0.0, force=False, model="bgk"):
    nx, ny, nz = shape
    m = np.zeros((nz, ny, nx), np.uint8)
    if solid == "walls":
        m[0] = m[-1] = 1
    elif solid:
        m = synthetic.random_mask3(nx, ny, nz, seed=7, solid_fraction=solid, walls=True)
    g = (2e-5, -1e-5, 1e-5) if force else (0.0, 0.0, 0.0)
    lat = lbm.Lattice3D(m, 0.7, force=g, dtype=dtype, layout=layout)
    if model == "mrt":
        lat.set_mrt(MRT)
    elif model == "trt":
        lat.set_trt(3.0 / 16.0)
    lat.init_equilibrium(*synthetic.random_fields3(nx, ny, nz, seed=8))
    return lat


def state(lat):
    import torch
    s = torch.zeros(lat.state_bytes(), dtype=torch.uint8, device="cuda")
    lat.save_state(s)
    return s


def both(lbm, counts, *args, **kw):
    """The raw state after each count of steps, taken as one call and one step at a time."""
    import torch
    a, b = make(lbm, *args, **kw), make(lbm, *args, **kw)
    for n in counts:
        a.step(n)
        for _ in range(n):
            b.step(1)
        assert torch.equal(state(a), state(b)), f"{args} {kw} after {n} steps"
    assert np.isfinite(a.mass())
    a.close()
    b.close()


@pytest.mark.parametrize("layout", ["dense_ab", "dense_aa"])
@pytest.mark.parametrize("shape", [(1, 130, 16), (31, 1, 2050), (64, 13, 158), (65, 2050, 1),
                                   (33, 27, 90), (129, 40, 18), (200, 12, 60), (32, 26, 79)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_sizes(lbm, dtype, shape, layout):
    announce(f"d3q19 pairs {shape} {dtype} {layout}")
    for walls in (0.0, "walls") if shape[2] > 2 else (0.0,):
        both(lbm, (2, 5, 4, 1, 6), shape, dtype, layout, solid=walls)


@pytest.mark.parametrize("layout", ["dense_ab", "dense_aa"])
@pytest.mark.parametrize("model", ["bgk", "trt", "mrt"])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_models(lbm, dtype, model, layout):
    announce(f"d3q19 pairs {model} {dtype} {layout}")
    for solid in (0.0, 0.15):
        for force in (False, True):
            both(lbm, (5, 4), (65, 66, 64), dtype, layout, solid=solid, force=force, model=model)


@pytest.mark.parametrize("layout", ["dense_ab", "dense_aa"])
@pytest.mark.parametrize("dtype,model", [("f16s", "bgk"), ("bf16s", "trt"), ("f16s", "mrt")])
def test_16_bit(lbm, dtype, model, layout):
    announce(f"d3q19 pairs {model} {dtype} {layout}")
    both(lbm, (3, 4), (129, 200, 185), dtype, layout, model=model)


@pytest.mark.parametrize("layout", ["dense_ab", "dense_aa"])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_state_between_pairs(lbm, dtype, layout):
    """The raw state after pairs is that of single steps and restarts both ways."""
    import torch
    announce(f"d3q19 pairs saved state {dtype} {layout}")
    args = ((65, 66, 64), dtype, layout, 0.1, True)
    a, b = make(lbm, *args), make(lbm, *args)
    a.step(5)
    for _ in range(5):
        b.step(1)
    sa, sb = state(a), state(b)
    assert torch.equal(sa, sb)
    a.step(6)
    want = a.get_populations()
    b.load_state(sa)
    b.step(6)
    a.load_state(sb)
    for _ in range(6):
        a.step(1)
    assert np.array_equal(b.get_populations(), want)
    assert np.array_equal(a.get_populations(), want)
    a.close()
    b.close()


@pytest.mark.parametrize("layout", ["dense_ab", "dense_aa"])
@pytest.mark.parametrize("n", [2, 4, 6])
def test_callers_graph(lbm, layout, n):
    """step(n) captured by the caller and replayed with eager steps in between: the graph finds
    the state where it was recorded."""
    import torch
    announce(f"d3q19 pairs captured {layout} {n}")
    args = ((70, 33, 32), "f32", layout, "walls")
    a, b = make(lbm, *args), make(lbm, *args)
    stream = torch.cuda.Stream()
    a.set_stream(stream)
    a.step(3)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        a.step(n)  # recorded, not run, and counted
    total = 3
    for eager in (2, 4, 6):
        with torch.cuda.stream(stream):
            graph.replay()
        a.step(eager)
        torch.cuda.synchronize()
        total += n + eager
    for _ in range(total):
        b.step(1)
    assert np.array_equal(a.get_populations(), b.get_populations())
    a.close()
    b.close()
