"""Several reverse steps per launch (the checkpointed driver on small lattices) against the
one-step entry points: dJ/dalpha bitwise, dJ/dg up to the order of its FP64 sum.  Sizes of
one node, around the 22, 24 and 26 nodes that a square writes, and of several squares; segment
lengths that leave every remainder; solid nodes, with and without a drag field."""
import numpy as np
import pytest

import synthetic
from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("nx,ny,T,K", [(1, 3, 4, 4), (5, 7, 9, 3), (22, 22, 11, 11), (23, 45, 7, 6),
                                       (200, 61, 23, 5), (641, 180, 13, 13), (700, 200, 17, 8),
                                       (1000, 251, 19, 7)])
@pytest.mark.parametrize("drag", [True, False])
def test_squares_equal_single_steps(nx, ny, T, K, dtype, drag):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_13241_amd as lbm
    announce(f"adjoint squares {nx}x{ny} {dtype} T={T} K={K} drag={drag}")
    rng = np.random.default_rng(nx + ny)
    m = synthetic.random_mask(nx, ny, seed=3, solid_fraction=0.1, walls=ny > 4)
    m[:, nx - 1] = 0
    alpha = rng.random((ny, nx)).astype(np.float32)

    def lattice():
        lat = lbm.Lattice(m, 0.8, force=(1e-4, -2e-4), dtype=dtype, layout="dense_ab")
        if drag:
            lat.set_porosity(alpha)
        lat.init_equilibrium(*synthetic.random_fields(nx, ny, seed=4, u_amp=0.03))
        return lat

    def grads():
        return (torch.zeros((ny, nx), dtype=torch.float64, device="cuda"),
                torch.zeros(2, dtype=torch.float64, device="cuda"))

    a = lattice()
    sb = a.state_bytes()
    ckpt = torch.empty(((T + K - 1) // K) * sb, dtype=torch.uint8, device="cuda")
    seg = torch.empty(K * sb, dtype=torch.uint8, device="cuda")
    ga, gg = grads()
    a.run_checkpointed(T, K, ckpt)
    a.adjoint_checkpointed(T, K, ckpt, seg, nx - 1, 1.0, ga, gg)

    b = lattice()
    states = torch.empty((T, sb), dtype=torch.uint8, device="cuda")
    for t in range(T):
        b.save_state(states[t])
        b.step(1)
    nb, _ = b.adjoint_bytes()
    mu = [torch.zeros(nb, dtype=torch.uint8, device="cuda") for _ in range(2)]
    gb, hb = grads()
    b.adjoint_seed_outlet_ux(nx - 1, 1.0, mu[0], gb, hb)
    terms = torch.zeros(2, dtype=torch.float64, device="cuda")
    for t in range(T - 1, -1, -1):
        k = (T - 1 - t) % 2
        before = hb.clone()
        b.adjoint_step(states[t], mu[k], mu[1 - k], gb, hb)
        terms += (hb - before).abs()
    torch.cuda.synchronize()
    assert torch.equal(ga, gb)
    # one FP64 sum of up to nx ny T terms in another order: each of about log2 levels rounds
    # by 2^-53 of sums no larger than the nodes' magnitudes, bounded by 64 ulps of their total
    scale = float(terms.abs().max()) + float(hb.abs().max())
    assert float((gg - hb).abs().max()) <= 64 * 2.0 ** -53 * max(scale, nx * ny * 1e-3)
    a.close()
    b.close()
