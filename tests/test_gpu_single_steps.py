"""The oracle tests of the single-step kernels, taken one step per call.

A call of several steps runs fused launches where those are faster, so tests written for the
single-step kernels (the LDS-staged segment kernels, the AA layout's even and odd steps, the
per-node kernels of small lattices, the tiled and listed ones) no longer launch them by calling
step(n) once.  Here the same tests run with every step a call of its own, which is one launch
of the kernel they name."""
import pytest

from test_gpu_d3q19 import (test_plane_channel_interior_segments,  # noqa: F401
                            test_random_solids_vs_oracle, test_trt_vs_oracle)
from test_gpu_d3q19_aa import test_aa_trt_and_force_free, test_aa_vs_oracle  # noqa: F401
from test_gpu_fullsize import (porous_mask, test_porous_4096,  # noqa: F401
                               test_taylor_green_4096_aa_odd, test_taylor_green_4096_bench_config)
from test_gpu_mrt import test_mrt_open_channel_vs_oracle, test_mrt_porous_vs_oracle  # noqa: F401
from test_gpu_mrt3 import test_mrt3_vs_oracle  # noqa: F401
from test_gpu_open import (test_channels_vs_oracle, test_lid_cavity_vs_oracle,  # noqa: F401
                           test_mixed_open_sides_force_drag)
from test_gpu_parity import (test_exact_rational_4x4, test_layouts_bitwise_equal,  # noqa: F401
                             test_porous_all_layouts_vs_oracle, test_ragged_shapes,
                             test_tiled_shapes)
from test_gpu_segment import (lbm, test_segment_kernel_16bit_bitwise,  # noqa: F401
                              test_segment_kernel_aa_vs_oracle, test_segment_kernel_mid_size,
                              test_segment_kernel_vs_oracle)
from test_gpu_segment3 import test_segment3_aa_vs_oracle, test_segment3_vs_oracle  # noqa: F401
from test_gpu_trt import test_trt_porous_vs_oracle  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def one_step_a_call(monkeypatch):
    import paper_2108_13241_amd as pkg

    for cls in (pkg.Lattice, pkg.Lattice3D):
        real = cls.step

        def step(self, n=1, real=real):
            for _ in range(n):
                real(self, 1)

        monkeypatch.setattr(cls, "step", step)
