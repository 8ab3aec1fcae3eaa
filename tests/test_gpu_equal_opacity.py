"""Frequencies of equal opacity ratio share one ray of the sweep (complete
redistribution): operator, right-hand side, diagonal, assembled matrix and
field against the oracle, which keeps every frequency, on grids with all,
some and none of the opacities equal.

Tolerances as in test_gpu_random and test_gpu_dense: 1e-12 normwise for the
FP64 operator, right-hand side and diagonal, 1e-5 for the FP32 operator, 1e-13
per matrix entry.  Merging replaces opacities that differ by at most 1e-12 by
their weighted mean, an error of second order (1e-24)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_2110_11873_amd import binding as B  # noqa: E402
from paper_2110_11873_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu

FS = ["delo_linear", "trapezoidal", "implicit_euler", "delo_parabolic"]


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).to("cuda")


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def _base(fs, ns=(40, 17), n_nu=21, normalize=True):
    return W.make_slabs(list(ns), [(1e-3, 1e5), (1e-2, 1e3)][:len(ns)], 6, n_nu, 5.0,
                        [1e-3, 5e-3][:len(ns)], [1e-2, 1e-1][:len(ns)], [0.5, 0.9][:len(ns)],
                        formal_solver=fs, normalize=normalize)


def _grid(kind, fs):
    """(problem, rays per direction that the sweep keeps)"""
    p = _base(fs, normalize=kind != "unnormalized")
    rng = np.random.default_rng(11)
    opac, phi, w = p.opac.copy(), p.phi.copy(), p.w_nu.copy()
    n = p.n_nu
    if kind in ("even", "unnormalized"):
        count = 11
    elif kind == "shifted":  # a profile that is not even: nothing to merge
        opac *= np.exp(0.02 * p.x)[None, :]
        count = n
    elif kind == "one slab shifted":  # different counts: the shorter one is padded
        opac[1] *= np.exp(0.02 * p.x)
        count = n
    elif kind == "constant":
        opac[:] = 0.3
        count = 1
    elif kind == "triples":  # in no order, with different weights
        opac[:] = rng.permutation(np.repeat(np.logspace(-3, 0, n // 3), 3))[None, :]
        count = n // 3
    elif kind == "no weight":  # merged groups without weight, alone and beside others
        w[[0, n - 1, 3]] = 0.0
        phi[1, 7] = phi[1, n - 8] = 0.0
        count = 11
    elif kind == "nearly":  # half of the pairs within 1e-12, half outside
        opac[:, n // 2 + 1:] = opac[:, :n // 2][:, ::-1]
        opac[:, :n // 2:2] *= 1 + 5e-13
        opac[:, 1:n // 2:2] *= 1 + 5e-12
        count = 16
    else:
        raise AssertionError(kind)
    return p.with_(opac=opac, phi=phi, w_nu=w), count


KINDS = ["even", "unnormalized", "shifted", "one slab shifted", "constant", "triples", "no weight",
         "nearly"]


@pytest.mark.parametrize("fs", FS)
@pytest.mark.parametrize("kind", KINDS)
def test_merged_rays_against_the_oracle(kind, fs):
    p, count = _grid(kind, fs)
    v = W.random_vector(p.n_unknowns, 3)
    ref = O.apply(p, v)
    scale = np.abs(v).max() + np.abs(v - ref).max()
    # a grid of `count` different opacities needs the same tiles
    alone = _base(fs, n_nu=max(count, 2))
    alone = alone.with_(opac=alone.opac * np.exp(0.02 * alone.x)[None, :])
    with B.setup(p, chunk=4) as h, B.setup(alone, chunk=4) as g:
        if count > 1:
            assert h.plan_info()["pairs"] == g.plan_info()["pairs"]
        assert np.abs(host(h.apply_op(dev(v))) - ref).max() <= 1e-12 * scale
        assert np.abs(host(h.apply_op_fp32(dev(v))) - ref).max() < 1e-5 * scale
        b, bref = host(h.get_rhs()), O.rhs(p)
        assert np.abs(b - bref).max() <= 1e-12 * np.abs(bref).max()
        idx = [0, 1, p.n_unknowns // 2, p.n_unknowns - 1]
        assert np.abs(host(h.get_jacobi_diag())[idx] - O.diag(p, idx)).max() <= 1e-12
        if fs != "delo_parabolic":
            A = h.assemble()
            for i, blk in enumerate(h.dense_blocks(A)):
                assert np.abs(host(blk) - O.assemble(p.slab(i))).max() <= 1e-13


@pytest.mark.parametrize("kind", ["even", "shifted", "triples"])
def test_field_keeps_every_frequency(kind):
    """The field has one intensity per frequency: J I + c of a random field by
    the quadrature over all of them."""
    p, _ = _grid(kind, "delo_linear")
    p = p.slab(0)
    rng = np.random.default_rng(5)
    n, mu = int(p.ns[0]), p.mu
    f = rng.uniform(-1.0, 1.0, (2, n, p.n_mu, p.n_nu))
    t1, t2 = np.sqrt(2) * (3 * mu ** 2 - 1) / 4, np.sqrt(2) * (3 * mu ** 2 - 3) / 4
    wp = p.w_nu * p.phi[0]
    q = 0.5 * p.w_mu[:, None] * (wp / wp.sum())[None, :]
    J0 = (q * f[0]).sum((1, 2))
    J2 = (q * (t1[:, None] * f[0] + t2[:, None] * f[1])).sum((1, 2))
    xi = 1 - p.eps[0]
    ref = np.stack([xi * J0 + p.eps[0] * p.B, xi * p.W2[0] * J2], 1).reshape(-1)
    with B.setup(p) as h:
        assert np.abs(host(h.sigma_from_field(dev(f.reshape(-1)))) - ref).max() <= 1e-13
