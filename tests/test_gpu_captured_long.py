"""Long calls captured by the caller: on contexts that would replay graphs of their own (small AA
lattices from 32 steps on; any with an explicit graph length), the caller's graph has to hold the
steps themselves.  Replayed several times with eager calls between, against single steps."""
import numpy as np
import pytest

import synthetic
from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout,graph,n", [("dense_aa", -1, 40), ("dense_aa", -1, 64),
                                            ("dense_aa", 10, 24), ("dense_ab", 10, 24),
                                            ("dense_ab", -1, 40), ("indirect", 2, 6)])
@pytest.mark.parametrize("warm", [0, 2])
def test_captured_long_calls(layout, graph, n, warm):
    """warm: own graphs exist already (an eager call of as many steps) or not."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_13241_amd as lbm
    announce(f"captured long call {layout} graphs of {graph}, {n} steps, warm={warm}")

    def make():
        m = synthetic.random_mask(150, 50, seed=5, solid_fraction=0.1, walls=True)
        lat = lbm.Lattice(m, 0.7, force=(2e-4, -1e-4), dtype="f32", layout=layout)
        lat.init_equilibrium(*synthetic.random_fields(150, 50, seed=6, u_amp=0.03))
        return lat

    a, b = make(), make()
    stream = torch.cuda.Stream()
    a.set_stream(stream)
    a.set_graph_steps(graph)
    total = 0
    for _ in range(warm):
        a.step(n)
        total += n
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        a.step(n)  # recorded, not run
    for eager in (2, n, 34):
        with torch.cuda.stream(stream):
            g.replay()
        a.step(eager)
        torch.cuda.synchronize()
        total += n + eager
        while total:
            b.step(1)
            total -= 1
        assert np.array_equal(a.get_populations(), b.get_populations()), eager
    a.close()
    b.close()
