"""Slabs that need chunks longer than 8, asked for with eight waves per block and
the chunk left to the library: eight waves are compiled for chunks up to 8
only, so the sweep runs with four.  One slab, a few, and enough that a block
holds several directions.  Tolerance 1e-12 normwise, as for the operator."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_2110_11873_amd import binding as B  # noqa: E402
from paper_2110_11873_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).to("cuda")


@pytest.mark.parametrize("n,deep,m,n_nu", [(1, 600, 5, 41), (3, 1100, 4, 23), (330, 530, 8, 17), (1300, 515, 4, 6)])
@pytest.mark.parametrize("fs", ["delo_linear", "delo_parabolic"])
def test_deep_slabs_with_eight_waves(n, deep, m, n_nu, fs):
    rng = np.random.default_rng(n)
    ns = [deep] + list(rng.integers(4, 20, n - 1))
    p = W.make_slabs(ns, [(1e-3, 10.0 ** e) for e in rng.uniform(2, 6, n)], 2 * m, n_nu, 4.0,
                     list(10.0 ** rng.uniform(-4, -2, n)), [1e-2] * n, [0.5] * n, formal_solver=fs)
    v = W.random_vector(p.n_unknowns, n)
    ref, b = O.apply(p, v), O.rhs(p)
    scale = np.abs(v).max() + np.abs(v - ref).max()
    with B.setup(p, sweep_waves=8, rtol=1e-10, maxit=20000) as h:
        assert h.plan_info()["chunk"] > 8
        assert np.abs(h.apply_op(dev(v)).cpu().numpy() - ref).max() <= 1e-12 * scale
        assert np.abs(h.apply_op_fp32(dev(v)).cpu().numpy() - ref).max() <= 1e-5 * scale
        assert np.abs(h.get_rhs().cpu().numpy() - b).max() <= 1e-12 * np.abs(b).max()
        assert h.sweep_config()["waves"] == 4
