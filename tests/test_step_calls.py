"""What Lattice.step costs beside the launch: calls of a few steps go straight to the library,
on the AA layout as well (its longer calls ask for memory to lend first)."""
import pytest

import paper_2108_13241_amd as lbm


class Recorder:
    def __init__(self):
        self.calls = []

    def __getattr__(self, name):
        def call(*args):
            self.calls.append(name)
            return 0
        return call


@pytest.mark.parametrize("cls,prefix", [(lbm.Lattice, "lbm"), (lbm.Lattice3D, "lbm3d")])
@pytest.mark.parametrize("layout", ["dense_ab", "dense_aa", "indirect"])
def test_few_steps_are_one_call(cls, prefix, layout):
    lat = cls.__new__(cls)
    lat.layout, lat.in_place, lat._ctx, lat._lib = layout, False, None, Recorder()
    for n in (0, 1, 2, 3):
        lat.step(n)
    assert lat._lib.calls == [f"{prefix}_step"] * 4


@pytest.mark.parametrize("cls", [lbm.Lattice, lbm.Lattice3D])
@pytest.mark.parametrize("n", ["5", 5.0, True])
def test_counts_are_taken_as_int_takes_them(cls, n):
    lat = cls.__new__(cls)
    lat.layout, lat.in_place, lat._ctx, lat._lib = "dense_aa", True, None, Recorder()
    lat.step(n)
    assert len(lat._lib.calls) == 1
