"""Waves per block of a single slab: eight only while each has an LDS row of its
own for its sums (455 points of 64 KB); the operator at the line, against the
oracle.  Tolerance 1e-12 normwise, as for the operator."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_2110_11873_amd import binding as B  # noqa: E402
from paper_2110_11873_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns,waves", [(200, 8), (455, 8), (456, 4), (512, 4), (513, 4)])
def test_waves_of_a_single_slab(ns, waves):
    p = W.make_slabs([ns], [(1e-4, 1e6)], 16, 33, 6.0, [1e-3], [1e-2], [0.5])
    v = W.random_vector(p.n_unknowns, ns)
    ref = O.apply(p, v)
    with B.setup(p) as h:
        assert h.sweep_config()["waves"] == waves
        y = h.apply_op(torch.from_numpy(v).cuda()).cpu().numpy()
    assert np.abs(y - ref).max() <= 1e-12 * (np.abs(v).max() + np.abs(v - ref).max())


@pytest.mark.parametrize("ns,m,waves,blocks", [(40, 4, 8, 1), (200, 10, 4, None), (512, 8, 4, None)])
def test_waves_of_a_single_parabolic_slab(ns, m, waves, blocks):
    """Four, but for a slab that one block of eight holds."""
    p = W.make_slabs([ns], [(1e-4, 1e6)], 2 * m, 21, 6.0, [1e-3], [1e-2], [0.5], formal_solver="delo_parabolic")
    v = W.random_vector(p.n_unknowns, ns)
    ref = O.apply(p, v)
    with B.setup(p) as h:
        assert h.sweep_config()["waves"] == waves
        assert blocks is None or h.plan_info()["blocks"] == blocks
        y = h.apply_op(torch.from_numpy(v).cuda()).cpu().numpy()
    assert np.abs(y - ref).max() <= 1e-12 * (np.abs(v).max() + np.abs(v - ref).max())
