"""Single slabs under options.graphs: one block that ends the operator itself, blocks
on one XCD, blocks on all, and FP32 sweeps with a plan of their own.  Replays give
what eager launches give, to the bit, with eager work between them; and the
operator captured by the caller."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2110_11873_amd import binding as B  # noqa: E402
from paper_2110_11873_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu

# slabs, depths, directions, frequencies, distinct opacities
SHAPES = [(1, 40, 4, 21, False), (1, 100, 4, 51, False), (1, 200, 10, 101, False), (1, 283, 8, 101, True),
          (1, 400, 16, 201, False), (1, 512, 8, 64, False), (1300, 20, 4, 9, True)]


def problem(n, ns, m, n_nu, distinct, fs):
    p = W.make_slabs([ns] * n, [(1e-3, 1e4)] * n, 2 * m, n_nu, 5.0, [1e-3] * n, [1e-2] * n, [0.5] * n, formal_solver=fs)
    return p.with_(opac=p.opac * (1 + 1e-3 * np.arange(n_nu))) if distinct else p


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s[:4])))
@pytest.mark.parametrize("fs", ["delo_linear", "delo_parabolic"])
@pytest.mark.parametrize("kind,mixed", [("gmres", False), ("gmres", True), ("bicgstab", False)])
def test_replays_give_the_eager_result(shape, fs, kind, mixed):
    p = problem(*shape, fs)
    kw = dict(rtol=1e-9, maxit=20000, precision=B.RT_PREC_MIXED if mixed else B.RT_PREC_FP64, check_every=8)
    x0 = torch.from_numpy(W.initial_guess(p)).cuda()
    v = torch.from_numpy(W.random_vector(p.n_unknowns, 1)).cuda()
    with B.setup(p, graphs=0, **kw) as h:
        ref, y0 = x0.clone(), h.apply_op(v)
        rc, info = getattr(h, "solve_" + kind)(ref)
        assert rc == 0
    with B.setup(p, graphs=1, **kw) as h:
        x = torch.empty_like(x0)
        for _ in range(3):
            assert torch.equal(h.apply_op(v), y0)
            torch.cuda.synchronize()
            x.copy_(x0)
            _, again = getattr(h, "solve_" + kind)(x)
            assert torch.equal(x, ref) and [i.iterations for i in again] == [i.iterations for i in info]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s[:4])))
def test_operator_captured_by_the_caller(shape):
    p = problem(*shape, "delo_linear")
    v = torch.from_numpy(W.random_vector(p.n_unknowns, 1)).cuda()
    with B.setup(p) as h:
        u, y, y32 = v.clone(), torch.empty_like(v), torch.empty_like(v)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            h.apply_op(u, y)
            h.apply_op_fp32(u, y32)
        for s in range(4):
            u.copy_(torch.from_numpy(W.random_vector(p.n_unknowns, s)))
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(y, h.apply_op(u)) and torch.equal(y32, h.apply_op_fp32(u))
