"""The FP32 operator adds the sums of different directions in FP64, also where
one block holds several directions.  Two |mu|, the second of weight 2^-12: the
first one's quadrature is exact in FP32 (implicit Euler steps of optical depth
1 halve numbers of few bits), so what is lost against the FP64 operator is the FP32
rounding of the second one's terms, some 2^-12 x 1e-7 of them, and not a rounding
of the sum, which an FP32 sum of the two would give (6e-8 of it)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2110_11873_amd import binding as B  # noqa: E402
from paper_2110_11873_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


# slabs, depths: one slab in one block; two directions per block of a batch,
# in rows of their own and (deep slabs) in one shared row of the block's LDS
@pytest.mark.parametrize("n,ns,deep", [(1, 5, 0), (1300, 5, 0), (1300, 5, 1700)])
def test_directions_are_added_in_fp64(n, ns, deep):
    depths = [ns] * n
    if deep:
        depths[0] = deep
    small = 2.0 ** -12
    p = W.make_slabs(depths, [(1.0, 2.0)] * n, 2, 2, 4.0, [1e-3] * n, [2.0 ** -6] * n, [0.5] * n, formal_solver="implicit_euler")
    p = p.with_(tau=np.concatenate([np.arange(1.0, d + 1) for d in depths]), mu=np.array([-1.0, -0.3, 0.3, 1.0]),
                w_mu=np.array([1 - small, small, small, 1 - small]), x=np.zeros(1), w_nu=np.ones(1),
                phi=np.ones((n, 1)), opac=np.ones((n, 1)))
    v = np.zeros(p.n_unknowns)
    v[0::2] = np.random.default_rng(3).integers(-8, 9, p.n_unknowns // 2)
    u = torch.from_numpy(v).cuda()
    with B.setup(p) as h:
        err = (h.apply_op_fp32(u) - h.apply_op(u))[0::2].abs().cpu().numpy()
    # sources up to 8, four terms of each direction; the deep slab only sets the block's LDS
    assert err[deep:].max() <= 8 * 4 * small * 1e-6


@pytest.mark.parametrize("n,m,n_nu,ns", [(1300, 4, 41, 30), (2700, 2, 23, 80), (700, 8, 9, 20)])
def test_waves_add_no_more_batches_in_fp32_than_with_a_ray_per_frequency(n, m, n_nu, ns):
    """Where no opacities are equal: the same sums, to the bit, as with all four
    waves of a block on one direction (a fixed number of batches per wave)."""
    p = W.make_slabs([ns] * n, [(1e-3, 1e4)] * n, 2 * m, n_nu, 4.0, [1e-3] * n, [1e-2] * n, [0.5] * n)
    p = p.with_(opac=p.opac * (1 + 1e-3 * np.arange(n_nu)))
    u = torch.from_numpy(W.random_vector(p.n_unknowns, n)).cuda()
    with B.setup(p) as h:
        y = h.apply_op_fp32(u)
        x = h.apply_op(u)
    with B.setup(p, wave_batches=32) as h:
        assert torch.equal(h.apply_op_fp32(u), y)
        assert (h.apply_op(u) - x).abs().max() <= 1e-12 * (u.abs().max() + (x - u).abs().max())
