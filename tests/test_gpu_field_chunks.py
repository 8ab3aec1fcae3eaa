"""The field operator's sweep at the edges of its chunks (4 points up to 256,
8 up to 512, the general kernel beyond), uneven slabs in one batch, workgroups
whose rays end mid-way, and a quadrature of more rays than its workgroup takes
in one turn, against the oracle.  Tolerance 1e-12 normwise, as in
test_gpu_field."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_2110_11873_amd import binding as B  # noqa: E402
from paper_2110_11873_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu

# depths of the slabs, directions, frequencies
CASES = [([2], 2, 3), ([31, 2, 32], 4, 5), ([33, 64], 6, 7), ([255], 4, 9), ([256, 129, 3], 2, 3),
         ([257], 4, 9), ([511, 17], 2, 5), ([512], 2, 3), ([513, 40], 2, 3), ([20], 32, 70)]


@pytest.mark.parametrize("fs", ["delo_linear", "trapezoidal", "implicit_euler"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, (*c[0], c[1], c[2]))))
def test_field_chunk_edges(case, fs):
    ns, n_mu, n_nu = case
    n = len(ns)
    p = W.make_slabs(ns, [(1e-3, 1e4)] * n, n_mu, n_nu, 4.0, [1e-3] * n, [1e-2] * n, [0.5] * n,
                     formal_solver=fs)
    rng = np.random.default_rng(3)
    with B.setup(p) as h:
        f = rng.uniform(-1, 1, h.field_size())
        y = h.apply_op_field(torch.from_numpy(f).cuda()).cpu().numpy()
        b = h.get_rhs_field().cpu().numpy()
    off = 0
    for i, k in enumerate(ns):
        q, m = p.slab(i), 2 * k * n_mu * n_nu
        order = lambda v: v[off:off + m].reshape(2, k, n_mu, n_nu).transpose(0, 2, 3, 1).ravel()  # noqa: B023,E731
        ref, rhs = O.apply_I(q, order(f)), O.rhs_I(q)
        scale = np.abs(f).max() + np.abs(order(f) - ref).max()
        assert np.abs(order(y) - ref).max() <= 1e-12 * scale
        assert np.abs(order(b) - rhs).max() <= 1e-12 * np.abs(rhs).max()
        off += m
