"""SOR with a NaN or an infinity in the vector: P = omega^-1 D + U is upper
triangular, so the unknowns after the bad one do not depend on it -- nor do they
in the block of 64 unknowns that holds it -- and stay what they were, to the
bit.  Sizes and places at the edges of the blocks."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2110_11873_amd import binding as B  # noqa: E402
from paper_2110_11873_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns,at", [(3, 2), (32, 0), (32, 40), (33, 64), (70, 10), (70, 63), (70, 64), (100, 130), (256, 300)])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_sor_keeps_the_unknowns_after_a_bad_one(ns, at, bad):
    p = W.make_slabs([ns], [(1e-3, 1e4)], 8, 9, 4.0, [1e-3], [1e-2], [0.5])
    v = W.random_vector(p.n_unknowns, ns)
    w = v.copy()
    w[at] = bad
    with B.setup(p, precond=B.RT_PC_SOR, omega=1.1) as h:
        x = h.precond_apply(torch.from_numpy(v).cuda()).cpu().numpy()
        y = h.precond_apply(torch.from_numpy(w).cuda()).cpu().numpy()
    assert np.array_equal(y[at + 1:], x[at + 1:]) and np.isfinite(x).all()
    assert not np.isfinite(y[at])
