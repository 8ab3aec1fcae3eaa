"""How the sweep's blocks share a slab: one, two or more waves per direction,
blocks of several directions (the last one partly empty where the directions
do not fill it), and several blocks per direction on a few slabs.  Operator in
both precisions, right-hand side and a mixed solve against the oracle.

Tolerances as in test_gpu_random: 1e-12 normwise in FP64, 1e-5 in FP32, the
solve below its rtol by the oracle's residual."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_2110_11873_amd import binding as B  # noqa: E402
from paper_2110_11873_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).to("cuda")


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


# slabs, directions (n_mu / 2), frequencies, deepest slab, waves per block,
# blocks: the directions of all slabs set the waves per direction (5120 waves
# in all are enough), and so the blocks per slab
PLANS = [(1280, 4, 3, 12, 4, 1280),       # one wave per direction, four directions per block
         (1800, 3, 4, 9, 4, 1800),        # ... of which the last wave has none
         (1280, 2, 3, 12, 4, 1280),       # two waves per direction, one of them without a batch
         (900, 3, 5, 40, 4, 1800),        # two blocks for three directions
         (640, 4, 3, 20, 8, 640),         # eight waves: two per direction
         (700, 5, 21, 70, 8, 1400),
         (5, 2, 61, 300, 4, None),        # a few slabs: blocks of two batches per wave
         (1, 7, 33, 513, 4, None)]


@pytest.mark.parametrize("plan", PLANS, ids=lambda p: "x".join(map(str, p)))
@pytest.mark.parametrize("fs", ["delo_linear", "trapezoidal", "delo_parabolic"])
def test_block_plans(plan, fs):
    n, m, n_nu, deepest, waves, blocks = plan
    rng = np.random.default_rng(n + m)
    ns = rng.integers(max(2, deepest // 4), deepest + 1, n)
    ns[0] = deepest
    p = W.make_slabs(list(ns), [(1e-3, 10.0 ** e) for e in rng.uniform(1, 5, n)], 2 * m, n_nu, 4.0,
                     list(10.0 ** rng.uniform(-4, -2, n)), list(10.0 ** rng.uniform(-2, -1, n)),
                     list(rng.uniform(0, 1, n)), formal_solver=fs)
    v = W.random_vector(p.n_unknowns, n)
    ref = O.apply(p, v)
    scale = np.abs(v).max() + np.abs(v - ref).max()
    with B.setup(p, precision=B.RT_PREC_MIXED, rtol=1e-9, sweep_waves=waves, maxit=20000) as h:
        assert blocks is None or h.plan_info()["blocks"] == blocks
        assert np.abs(host(h.apply_op(dev(v))) - ref).max() <= 1e-12 * scale
        assert np.abs(host(h.apply_op_fp32(dev(v))) - ref).max() < 1e-5 * scale
        b = O.rhs(p)
        assert np.abs(host(h.get_rhs()) - b).max() <= 1e-12 * np.abs(b).max()
        x = dev(W.initial_guess(p))
        rc, _ = h.solve_gmres(x)
        assert rc == 0
        r = b - O.apply(p, host(x))
        for s in O._slices(p):
            assert np.linalg.norm(r[s]) < 1e-9 * np.linalg.norm(b[s])


# depths, directions, frequencies of one slab; whether one block holds it
SINGLE = [(40, 4, 21, True), (2, 1, 2, True), (33, 8, 13, True), (256, 8, 3, True), (17, 5, 9, True),
          (65, 2, 31, True), (40, 9, 21, False), (200, 10, 101, False)]


@pytest.mark.parametrize("shape", SINGLE, ids=lambda s: "x".join(map(str, s[:3])))
@pytest.mark.parametrize("fs", ["delo_linear", "implicit_euler", "delo_parabolic"])
def test_one_slab(shape, fs):
    """One slab: in one block, which ends the operator itself, or in several
    blocks on one XCD; the same result in place and with the partial sums in
    the library's array."""
    ns, m, n_nu, whole = shape
    p = W.make_slabs([ns], [(1e-3, 1e4)], 2 * m, n_nu, 4.0, [1e-3], [1e-2], [0.5],
                     formal_solver=fs)
    v = W.random_vector(p.n_unknowns, ns)
    ref = O.apply(p, v)
    scale = np.abs(v).max() + np.abs(v - ref).max()
    with B.setup(p, rtol=1e-10, maxit=20000) as h:
        assert (h.plan_info()["blocks"] == 1) == whole
        y = h.apply_op(dev(v))
        assert np.abs(host(y) - ref).max() <= 1e-12 * scale
        x = dev(v)
        assert torch.equal(h.apply_op(x, x), y)
        if fs != "delo_parabolic":
            assert torch.equal(h.apply_op_noalloc(dev(v)), y)
        assert np.abs(host(h.apply_op_fp32(dev(v))) - ref).max() < 1e-5 * scale
        b = O.rhs(p)
        assert np.abs(host(h.get_rhs()) - b).max() <= 1e-12 * np.abs(b).max()
        for solve in (h.solve_gmres, h.solve_bicgstab):
            x = dev(W.initial_guess(p))
            rc, _ = solve(x)
            assert rc == 0
            r = b - O.apply(p, host(x))
            assert np.linalg.norm(r) < 2e-10 * np.linalg.norm(b)
