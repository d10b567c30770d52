"""A lattice that does not fit is refused and leaves no error behind: HIP keeps the last error of
a thread, and the next launch of any other lattice would report it as its own."""
import numpy as np
import pytest

import synthetic
from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [2, 3])
def test_refused_lattice_leaves_no_error(dims):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_13241_amd as lbm
    announce(f"refused lattice, {dims} dimensions")
    if dims == 2:
        def make(n):
            return lbm.Lattice(synthetic.all_fluid(n, n), 0.8, dtype="f64", torch_memory=False)
        small, big = 64, 9216  # 12 GB
    else:
        def make(n):
            return lbm.Lattice3D(np.zeros((n, n, n), np.uint8), 0.8, dtype="f64",
                                 torch_memory=False)
        small, big = 16, 384  # 17 GB
    lat = make(small)
    torch.cuda.empty_cache()
    free, _ = torch.cuda.mem_get_info()
    hold = torch.empty(free - (6 << 30), dtype=torch.uint8, device="cuda")
    with pytest.raises(lbm.LbmError) as e:
        make(big)
    assert e.value.status == -2
    lat.step(1)
    lat.step(4)
    assert abs(lat.mass() - small ** dims) < 1e-9 * small ** dims
    del hold
    torch.cuda.empty_cache()
    lat.close()
