"""Triangular solves (SOR, SSOR, LU) at the edges of their 64-unknown blocks:
one block and less, blocks that end exactly and one pair past the end, more
blocks than wavefronts, and a batch of more slabs than fit the chip at once
(the workgroup order).  Reference: the same substitutions in LAPACK on the
library's assembled A.  Tolerance 1e-11 of the largest value: the matrices
(eps 0.1 to 0.5) have condition numbers below 1e3, 64-bit substitution loses
at most N eps kappa ~ 1e-10 of the smallest and far less of the largest."""
import numpy as np
import pytest
from scipy.linalg import solve_triangular

torch = pytest.importorskip("torch")

from paper_2110_11873_amd import binding as B  # noqa: E402
from paper_2110_11873_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu

BATCHES = {"edges": [2, 3, 31, 32, 33, 63, 64, 65, 96, 97, 128],
           "deep": [545, 300, 257],
           "many": [2 + (7 * i) % 83 for i in range(531)]}


def _problem(ns):
    rng = np.random.default_rng(len(ns))
    n = len(ns)
    return W.make_slabs(ns, [(1e-3, 10.0 ** e) for e in rng.uniform(1, 4, n)], 4, 7, 4.0,
                        list(10.0 ** rng.uniform(-4, -2, n)), list(rng.uniform(0.1, 0.5, n)),
                        list(rng.uniform(0, 1, n)))


@pytest.mark.parametrize("batch", list(BATCHES))
@pytest.mark.parametrize("kind", ["sor", "ssor", "lu"])
def test_substitution(batch, kind):
    p = _problem(BATCHES[batch])
    v = W.random_vector(p.n_unknowns, 8)
    dv = torch.from_numpy(v).cuda()
    om = 1.3
    kw = {} if kind == "lu" else dict(
        precond=B.RT_PC_SOR if kind == "sor" else B.RT_PC_SSOR, omega=om)
    with B.setup(p, **kw) as h:
        blocks = [b.cpu().numpy() for b in h.dense_blocks(h.assemble())]
        if kind == "lu":
            x = torch.empty_like(dv)
            rc, _ = h.solve_lu(x, b=dv)
            assert rc == 0
        else:
            x = h.precond_apply(dv)
        x = x.cpu().numpy()
    off = 0
    for A in blocks:
        n = A.shape[0]
        b, got = v[off:off + n], x[off:off + n]
        off += n
        D = np.diag(np.diag(A))
        if kind == "lu":
            ref = np.linalg.solve(A, b)
        else:
            ref = solve_triangular(D / om + np.triu(A, 1), b, lower=False)
            if kind == "ssor":
                ref = solve_triangular(D / om + np.tril(A, -1), np.diag(A) * ref, lower=True)
                ref *= (2 - om) / om
        assert np.abs(got - ref).max() <= 1e-11 * np.abs(ref).max(), n
