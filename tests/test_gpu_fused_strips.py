"""The marching strips of the fused steps at the edges of their shape: lattices narrower than a
strip and around a multiple of what one writes (48, 56, 112 and 120 columns), of one and two rows,
in every layout and type; the collisions and boundaries of workloads that only large lattices
run; D3Q19 pairs on AA lattices large enough for them.  Each case first asks the library how
many steps its launches take, so that a changed threshold cannot leave it comparing single steps
with single steps."""
import numpy as np
import pytest

import fused_rules
import synthetic
from gpu_util import announce

pytestmark = pytest.mark.gpu

DTYPE = {"f64": 0, "f32": 1, "f16s": 2, "bf16s": 3}
LAYOUT = {"dense_ab": 0, "dense_aa": 1, "tiled16": 2, "indirect": 3}


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    return fused_rules.build(tmp_path_factory.mktemp("rules"))


def make(nx, ny, dtype, variant, layout, solid):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_13241_amd as lbm
    kinds = variant.split("+")
    m = synthetic.random_mask(nx, ny, seed=11, solid_fraction=solid, walls=ny > 4)
    g = (2e-4, -1e-4) if "force" in kinds or "drag" in kinds else (0.0, 0.0)
    lat = lbm.Lattice(m, 0.7, force=g, dtype=dtype, layout=layout)
    rng = np.random.default_rng(11)
    if "drag" in kinds:
        lat.set_porosity(rng.random((ny, nx)).astype(np.float32))
    if "open" in kinds:
        bc = np.zeros((ny, nx), dtype=np.uint8)
        val = np.zeros((2, ny, nx))
        bc[:, 0], bc[:, -1] = 5, 6
        bc[m != 0] = 0
        val[0] = np.where(bc >= 5, 1.0 + 0.01 * rng.random((ny, nx)), 0.0)
        lat.set_boundaries(bc, val)
    if "trt" in kinds:
        lat.set_trt(3.0 / 16.0)
    if "mrt" in kinds:
        lat.set_mrt((1.64, 1.54, 1.9))
    lat.init_equilibrium(*synthetic.random_fields(nx, ny, seed=12, u_amp=0.03))
    return lat


def check(driver, nx, ny, dtype, variant, layout, counts, solid=0.05):
    import torch
    announce(f"strips {nx}x{ny} {dtype} {layout} {variant} {counts}")
    a, b = (make(nx, ny, dtype, variant, layout, solid) for _ in range(2))
    kinds = variant.split("+")
    drag, coll = "drag" in kinds, 1 if "trt" in kinds else 2 if "mrt" in kinds else 0
    case = (nx, ny, DTYPE[dtype], LAYOUT[layout], int(drag or "force" in kinds), int(drag),
            int("open" in kinds), coll, a.info()["n_fluid"] / (nx * ny))
    (most, _), = fused_rules.ask(driver, [(*case, 100)])
    assert most >= 6, most  # strips take six or eight steps a launch
    sa, sb = (torch.zeros(a.state_bytes(), dtype=torch.uint8, device="cuda") for _ in range(2))
    for n in counts:
        a.step(n)
        for _ in range(n):
            b.step(1)
        a.save_state(sa)
        b.save_state(sb)
        assert torch.equal(sa, sb), n
    assert np.isfinite(a.mass())
    a.close()
    b.close()


# widths below, at and past one and two strips, and the heights that leave the squares for them
NARROW = [1, 2, 47, 48, 49, 55, 56, 57, 96, 112, 113, 120, 121, 240]


@pytest.mark.parametrize("dtype", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("nx", NARROW)
def test_narrow(driver, nx, dtype):
    wide = (nx + 23) // 24  # squares across
    ny = 24 * ((513 if dtype == "f64" else 1501) // wide + 2) + 5
    check(driver, nx, ny, dtype, "force", "dense_ab", (11, 3))


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("layout", ["dense_aa", "indirect"])
@pytest.mark.parametrize("nx", [47, 56, 113, 121])
def test_narrow_other_layouts(driver, nx, layout, dtype):
    wide = (nx + 23) // 24
    ny = 24 * ((513 if dtype == "f64" else 1501) // wide + 2) + 5
    check(driver, nx, ny, dtype, "force", layout, (11, 9))


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("nx", [16, 48, 112, 128])
def test_narrow_tiled(driver, nx, dtype):
    wide = (nx + 23) // 24
    ny = 16 * ((24 * ((513 if dtype == "f64" else 1501) // wide + 2) + 16) // 16)
    check(driver, nx, ny, dtype, "force", "tiled16", (11, 9))


@pytest.mark.parametrize("layout", ["tiled16", "tiled16_all"])
@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16s"])
@pytest.mark.parametrize("counts", [(8,), (6,), (1, 8), (4, 4, 5), (11, 1)])
def test_raw_state_of_tiles(dtype, layout, counts):
    """Saved states of tiles hold solid slots too: those of single steps, however the steps were
    grouped, after an initialisation, a re-initialisation and a loaded state."""
    import torch
    announce(f"raw state of tiles {dtype} {layout} {counts}")
    a, b = (make(160, 48, dtype, "force", layout, 0.2) for _ in range(2))
    sa, sb, s0 = (torch.zeros(a.state_bytes(), dtype=torch.uint8, device="cuda") for _ in range(3))
    a.save_state(s0)
    for start in ("fields", "rest", "loaded"):
        if start == "rest":
            a.init_equilibrium()
            b.init_equilibrium()
        elif start == "loaded":
            a.load_state(s0)
            b.load_state(s0)
        for n in counts:
            a.step(n)
            for _ in range(n):
                b.step(1)
            a.save_state(sa)
            b.save_state(sb)
            assert torch.equal(sa, sb), (start, n)
    a.close()
    b.close()


@pytest.mark.parametrize("layout", ["dense_ab", "dense_aa", "indirect"])
@pytest.mark.parametrize("ny", [1, 2, 3])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_low(driver, dtype, ny, layout):
    check(driver, 40011, ny, dtype, "force", layout, (11, 9))


@pytest.mark.parametrize("dtype", ["f16s", "bf16s"])
@pytest.mark.parametrize("ny", [1, 2])
def test_low_16_bit(driver, dtype, ny):
    check(driver, 40011, ny, dtype, "force", "dense_ab", (11, 9))


@pytest.mark.parametrize("layout", ["dense_ab", "dense_aa", "indirect", "tiled16"])
@pytest.mark.parametrize("variant", ["mrt+force", "drag", "drag+trt", "drag+mrt", "open+mrt+force",
                                     "open+drag"])
def test_fp32_variants(driver, variant, layout):
    check(driver, 1216, 912, "f32", variant, layout, (13, 8), solid=0.03)


@pytest.mark.parametrize("layout", ["dense_ab", "dense_aa"])
@pytest.mark.parametrize("variant,size", [("drag", (1216, 912)), ("trt+force", (1216, 912)),
                                          ("open+force", (2560, 2400)), ("mrt", (2560, 2400))])
def test_bf16_variants(driver, variant, size, layout):
    check(driver, *size, "bf16s", variant, layout, (13,), solid=0.01)


@pytest.mark.parametrize("variant", ["mrt+force", "drag+mrt", "open+mrt+force", "trt+force"])
@pytest.mark.parametrize("layout", ["dense_ab", "dense_aa", "indirect", "tiled16"])
def test_fp64_variants(driver, variant, layout):
    check(driver, 1216, 912, "f64", variant, layout, (13, 8))


@pytest.mark.parametrize("model", ["bgk", "trt", "mrt"])
@pytest.mark.parametrize("dtype,force", [("f32", False), ("f32", True), ("f64", True)])
@pytest.mark.parametrize("layout", ["dense_ab", "dense_aa"])
def test_pairs_with_solids(driver, layout, dtype, force, model):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_13241_amd as lbm
    nx, ny, nz = 65, 67, 130
    announce(f"d3q19 pairs {nx}x{ny}x{nz} {dtype} {layout} {model} force={force}")
    m = synthetic.random_mask3(nx, ny, nz, seed=7, solid_fraction=0.15, walls=True)
    fluid = float((m == 0).mean())
    if not (dtype == "f32" and model == "mrt" and force):  # single steps are faster there
        assert fused_rules.ask(driver, [(nx, ny, nz, DTYPE[dtype], int(layout == "dense_aa"),
                                         int(force), fluid)], "3") == [[1]]

    def make3():
        lat = lbm.Lattice3D(m, 0.7, force=(2e-5, -1e-5, 1e-5) if force else (0.0, 0.0, 0.0),
                            dtype=dtype, layout=layout)
        if model == "mrt":
            lat.set_mrt((1.19, 1.4, 1.64, 1.3, 1.55))
        elif model == "trt":
            lat.set_trt(3.0 / 16.0)
        lat.init_equilibrium(*synthetic.random_fields3(nx, ny, nz, seed=8))
        return lat

    a, b = make3(), make3()
    sa, sb = (torch.zeros(a.state_bytes(), dtype=torch.uint8, device="cuda") for _ in range(2))
    for n in (5, 4, 6):
        a.step(n)
        for _ in range(n):
            b.step(1)
        a.save_state(sa)
        b.save_state(sb)
        assert torch.equal(sa, sb), n
    a.close()
    b.close()
