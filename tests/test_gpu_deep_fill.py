"""Slabs whose chunks are longer than 8: where their directions leave room for it,
the blocks (one per CU at a time in FP64) number at most one per CU and one more
per direction for the remainders.  The operator of one such plan against the
oracle, 1e-12 normwise."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_2110_11873_amd import binding as B  # noqa: E402
from paper_2110_11873_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,ns,m,n_nu", [(1, 1024, 16, 201), (3, 1000, 8, 101), (8, 600, 8, 101), (1, 515, 3, 7), (2, 2000, 4, 33)])
def test_blocks_of_deep_slabs(n, ns, m, n_nu):
    rng = np.random.default_rng(n)
    p = W.make_slabs([ns] * n, [(1e-4, 10.0 ** e) for e in rng.uniform(3, 7, n)], 2 * m, n_nu, 6.0, [1e-3] * n, [1e-2] * n, [0.5] * n)
    p = p.with_(opac=p.opac * (1 + 1e-3 * np.arange(n_nu)))  # every opacity its own ray
    v = W.random_vector(p.n_unknowns, n)
    with B.setup(p) as h:
        assert h.plan_info()["chunk"] > 8
        assert h.plan_info()["blocks"] <= 256 + n * m
        y = h.apply_op(torch.from_numpy(v).cuda()).cpu().numpy()
    s = slice(0, 2 * ns)
    ref = O.apply(p.slab(0), v[s].copy())
    assert np.abs(y[s] - ref).max() <= 1e-12 * (np.abs(v[s]).max() + np.abs(v[s] - ref).max())
