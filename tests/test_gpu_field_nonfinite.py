"""A field with a NaN or an infinity at a slab's first or last depth.  The rays
that enter the slab there carry the boundary value, whatever the source at that
depth: the operator returns their input as it is, to the bit.  Depths at the
remainders of the sweep's chunks of 4 and 8 points."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2110_11873_amd import binding as B  # noqa: E402
from paper_2110_11873_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns", [2, 31, 64, 200, 256, 300, 512, 600])
@pytest.mark.parametrize("fs", ["delo_linear", "trapezoidal", "implicit_euler", "delo_parabolic"])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_boundary_values_do_not_see_the_source(ns, fs, bad):
    p = W.make_slabs([ns], [(1e-3, 1e4)], 8, 9, 4.0, [1e-3], [1e-2], [0.5], formal_solver=fs)
    f = np.random.default_rng(ns).uniform(-1, 1, (2, ns, 8, 9))
    entering = {0: p.mu < 0, ns - 1: p.mu > 0}  # depth: the directions that enter there
    with B.setup(p) as h:
        for k, rays in entering.items():
            g = f.copy()
            g[0, k, np.flatnonzero(~rays)[0], 4] = bad  # in a ray that leaves there
            y = h.apply_op_field(torch.from_numpy(g.ravel()).cuda()).cpu().numpy().reshape(f.shape)
            assert np.array_equal(y[:, k, rays], f[:, k, rays])
