"""Several steps per launch give bitwise the state of as many single steps, in every layout.

A call of one step runs the single-step kernels, which the other tests pin to the oracle; a
call of n > 1 steps runs the fused kernel.  Sizes sit at the edges of its strips (48, 56, 112
and 120 columns), below one strip and one row, and above several strips; step counts cover
every number of steps per launch and uneven splits.  Lattices of up to about 500^2 nodes run
the fused steps on squares, larger ones on strips.
"""
import numpy as np
import pytest

from gpu_util import announce

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (5, 3), (48, 17), (57, 2), (111, 9), (112, 40), (113, 33), (241, 26), (500, 75),
         (1, 5000), (7, 9000), (30011, 9), (1009, 601)]
DTYPES = ["f64", "f32", "f16s", "bf16s"]


def _lattice(nx, ny, dtype, variant, seed, layout="dense_ab", solid=0.1):
    import paper_2108_13241_amd as lbm
    import synthetic
    kinds = variant.split("+")
    walls = "solid" in kinds
    m = (synthetic.random_mask(nx, ny, seed=seed, solid_fraction=solid, walls=ny > 4)
         if walls else synthetic.all_fluid(nx, ny))
    g = (2e-4, -1e-4) if "force" in kinds or "drag" in kinds else (0.0, 0.0)
    lat = lbm.Lattice(m, 0.7, force=g, dtype=dtype, layout=layout)
    rng = np.random.default_rng(seed)
    if "drag" in kinds:
        lat.set_porosity(rng.random((ny, nx)).astype(np.float32))
    if "open" in kinds:
        bc = np.zeros((ny, nx), dtype=np.uint8)
        val = np.zeros((2, ny, nx))
        bc[:, 0], bc[:, -1] = 5, 6
        if ny > 2:
            bc[-1, 1:-1] = 4
        bc[m != 0] = 0
        val[0] = np.where(bc >= 5, 1.0 + 0.01 * rng.random((ny, nx)), 0.02)
        lat.set_boundaries(bc, val)
    if "trt" in kinds:
        lat.set_trt(3.0 / 16.0)
    if "mrt" in kinds:
        lat.set_mrt((1.64, 1.54, 1.9))
    lat.init_equilibrium(*synthetic.random_fields(nx, ny, seed=seed + 1, u_amp=0.03))
    return lat, m


def _check(nx, ny, dtype, variant, counts, seed=11, layout="dense_ab"):
    announce(f"fused steps {nx}x{ny} {dtype} {layout} {variant} {counts}")
    fused, m = _lattice(nx, ny, dtype, variant, seed, layout)
    single, _ = _lattice(nx, ny, dtype, variant, seed, layout)
    for n in counts:
        fused.step(n)
        for _ in range(n):
            single.step(1)
        a, b = fused.get_populations(), single.get_populations()
        assert np.isfinite(b[:, m == 0]).all()
        assert np.array_equal(a, b), (n, np.abs(a - b).max())
    fused.close()
    single.close()


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("nx,ny", SIZES)
def test_sizes(nx, ny, dtype):
    _check(nx, ny, dtype, "solid+force", [2, 8, 5])


# squares of 16 and 32 nodes at each number of steps, and strips, with a ragged rest
@pytest.mark.parametrize("layout", ["dense_ab", "dense_aa", "indirect"])
@pytest.mark.parametrize("dtype", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("nx,ny", [(129, 121), (250, 241), (285, 283), (321, 309), (351, 347),
                                   (530, 527), (611, 590)])
def test_square_sizes(nx, ny, dtype, layout):
    _check(nx, ny, dtype, "solid+force", [9, 8, 4], layout=layout)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("variant", ["", "trt", "mrt", "force", "solid", "solid+trt+force",
                                     "solid+mrt+force", "solid+drag", "solid+drag+trt",
                                     "solid+drag+mrt", "open", "open+trt", "open+mrt+force",
                                     "open+solid+drag+mrt"])
def test_variants(variant, dtype):
    _check(131, 37, dtype, variant, [7, 9])
    if dtype in ("f64", "f32"):
        _check(1031, 577, dtype, variant, [11])


@pytest.mark.parametrize("layout", ["dense_ab", "dense_aa", "indirect"])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_step_counts(dtype, layout):
    _check(150, 50, dtype, "solid", list(range(1, 18)), layout=layout)


@pytest.mark.parametrize("layout", ["dense_aa", "indirect"])
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("nx,ny", SIZES)
def test_sizes_other_layouts(nx, ny, dtype, layout):
    _check(nx, ny, dtype, "solid+force", [3, 8, 5], layout=layout)


@pytest.mark.parametrize("layout", ["tiled16", "tiled16_all"])
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("nx,ny", [(16, 16), (48, 32), (112, 48), (128, 16), (336, 80), (1008, 608)])
def test_sizes_tiled(nx, ny, dtype, layout):
    _check(nx, ny, dtype, "solid+force", [3, 8, 5], layout=layout)


@pytest.mark.parametrize("layout", ["dense_aa", "indirect", "tiled16"])
@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16s"])
@pytest.mark.parametrize("variant", ["", "trt", "mrt", "force", "solid", "solid+trt+force",
                                     "solid+drag", "solid+drag+mrt", "open", "open+solid+trt",
                                     "open+solid+drag+mrt"])
def test_variants_other_layouts(variant, dtype, layout):
    _check(144, 48, dtype, variant, [7, 10], layout=layout)
    if dtype != "bf16s":
        _check(1072, 592, dtype, variant, [11], layout=layout)


@pytest.mark.parametrize("layout", ["indirect", "tiled16"])
def test_sparse_holes(layout):
    """Whole solid squares, rows and strips between the fluid nodes, and one fluid node."""
    import paper_2108_13241_amd as lbm
    announce(f"fused steps, sparse holes, {layout}")
    m = np.ones((960, 640), dtype=np.uint8)
    m[100:900, :] = 0
    m[20:45, 30:90] = 0
    m[60:75, 150:320] = 0
    m[300:420, 100:500] = 1
    m[350, 200] = 0
    m[0:3, :40] = 0
    lats = [lbm.Lattice(m, 0.8, force=(1e-4, 2e-4), dtype="f64", layout=layout) for _ in range(2)]
    lats[0].step(23)
    for _ in range(23):
        lats[1].step(1)
    a, b = (lat.get_populations() for lat in lats)
    assert np.array_equal(a, b)


@pytest.mark.parametrize("layout", ["dense_ab", "dense_aa"])
@pytest.mark.parametrize("graph", [0, 2, 10, 34])
def test_graph_lengths(graph, layout):
    """Replays of any even length return to the lattice they start from."""
    announce(f"fused steps, graphs of {graph}, {layout}")
    fused, _ = _lattice(200, 60, "f32", "solid+force", 5, layout)
    single, _ = _lattice(200, 60, "f32", "solid+force", 5, layout)
    fused.set_graph_steps(graph)
    for n in (35, 1, 69, 14, 36):
        fused.step(n)
        for _ in range(n):
            single.step(1)
        assert np.array_equal(fused.get_populations(), single.get_populations())


def test_save_state_between_groups():
    """The raw state after a fused call is that of single steps (solid slots included)."""
    import torch
    announce("fused steps, raw state")
    fused, _ = _lattice(150, 50, "f64", "solid", 3)
    single, _ = _lattice(150, 50, "f64", "solid", 3)
    fused.step(13)
    for _ in range(13):
        single.step(1)
    n = fused.state_bytes()
    a = torch.zeros(n, dtype=torch.uint8, device="cuda")
    b = torch.zeros(n, dtype=torch.uint8, device="cuda")
    fused.save_state(a)
    single.save_state(b)
    assert torch.equal(a, b)


@pytest.mark.parametrize("layout", ["dense_ab", "dense_aa", "indirect"])
@pytest.mark.parametrize("n", [2, 8, 14])
def test_callers_graph(layout, n):
    """A caller's graph of step(n), replayed with eager calls of an even number of steps between
    the replays: it finds the state where it was recorded."""
    import torch
    announce(f"fused steps, captured by the caller, {layout} {n}")
    a, _ = _lattice(150, 50, "f32", "solid+force", 5, layout)
    b, _ = _lattice(150, 50, "f32", "solid+force", 5, layout)
    stream = torch.cuda.Stream()
    a.set_stream(stream)
    a.step(9)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        a.step(n)  # recorded, not run, and counted
    total = 9
    for eager in (8, 2, 22):
        with torch.cuda.stream(stream):
            graph.replay()
        a.step(eager)
        torch.cuda.synchronize()
        total += n + eager
    for _ in range(total):
        b.step(1)
    assert np.array_equal(a.get_populations(), b.get_populations())


def _check_state(nx, ny, dtype, variant, layout, counts, solid=0.05):
    import torch
    announce(f"fused steps {nx}x{ny} {dtype} {layout} {variant} {counts}")
    fused, _ = _lattice(nx, ny, dtype, variant, 21, layout, solid)
    single, _ = _lattice(nx, ny, dtype, variant, 21, layout, solid)
    a, b = (torch.zeros(fused.state_bytes(), dtype=torch.uint8, device="cuda") for _ in range(2))
    for n in counts:
        fused.step(n)
        for _ in range(n):
            single.step(1)
        fused.save_state(a)
        single.save_state(b)
        assert torch.equal(a, b), n
    fused.close()
    single.close()


@pytest.mark.parametrize("layout", ["dense_ab", "dense_aa", "indirect", "tiled16"])
@pytest.mark.parametrize("variant", ["solid+force", "solid+trt", "solid+mrt", "solid+drag", "open"])
@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16s"])
def test_strips(dtype, variant, layout):
    """Lattices just beyond those that run on squares."""
    if layout == "dense_aa" and "drag" in variant:
        variant = "force"
    _check_state(1216, 912, dtype, variant, layout, (13, 8))
    if layout != "tiled16":
        _check_state(40011, 9, dtype, variant, layout, (9,))


@pytest.mark.parametrize("layout,variant", [("indirect", "solid+force"), ("tiled16", "solid"),
                                            ("dense_ab", "mrt"), ("dense_aa", "open")])
@pytest.mark.parametrize("dtype", ["f16s", "bf16s"])
def test_large_16_bit(dtype, layout, variant):
    """The 16-bit variants that only large lattices run on strips."""
    _check_state(2560, 2400, dtype, variant, layout, (11,))


def test_second_lattice_belongs_to_its_stream(monkeypatch):
    """The AA layout's second lattice is allocated on the lattice's stream, whatever stream is
    current where step is called."""
    import torch
    announce("fused steps, AA on a stream of its own")
    side = torch.cuda.Stream()
    fused, _ = _lattice(150, 50, "f32", "solid+force", 5, "dense_aa")
    single, _ = _lattice(150, 50, "f32", "solid+force", 5, "dense_aa")
    fused.set_stream(side)
    seen, real = [], torch.empty

    def empty(*args, **kwargs):
        seen.append(torch.cuda.current_stream())
        return real(*args, **kwargs)

    monkeypatch.setattr(torch, "empty", empty)
    fused.step(9)
    monkeypatch.undo()
    assert seen and all(s == side for s in seen)
    for _ in range(9):
        single.step(1)
    assert np.array_equal(fused.get_populations(), single.get_populations())
