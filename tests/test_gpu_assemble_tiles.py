"""The assembly's tiles of 16 depths and blocks of 64 columns at their edges,
every compiled number of rays per wavefront, chunks of one |mu| over several
wavefronts, and rays over several slices, against the oracle's column-by-column
assembly.  Tolerance 1e-13 per entry, as in test_gpu_dense: sums of
nonnegative-weighted intensities bounded by one, in FP64."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_2110_11873_amd import binding as B  # noqa: E402
from paper_2110_11873_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu

EDGES = [2, 3, 15, 16, 17, 31, 33, 63, 64, 65, 79, 81, 128, 130]
# (n_mu / 2, different opacities): ray slots per wavefront 8, 16, 28, 40, 52
# (full and not), two wavefronts per |mu|, two slices with an empty wavefront
RAYS = [(2, 8), (8, 9), (3, 17), (4, 28), (1, 40), (2, 41), (8, 52), (3, 53), (9, 30), (5, 61)]


def _check(p):
    with B.setup(p) as h:
        A = h.assemble()
        torch.cuda.synchronize()
        for i, blk in enumerate(h.dense_blocks(A)):
            got = blk.cpu().numpy()
            ref = O.assemble(p.slab(i))
            assert np.abs(got - ref).max() <= 1e-13, int(p.ns[i])


@pytest.mark.parametrize("fs", ["delo_linear", "trapezoidal", "implicit_euler"])
def test_tile_edges(fs):
    n = len(EDGES)
    rng = np.random.default_rng(1)
    p = W.make_slabs(EDGES, [(1e-3, 10.0 ** e) for e in rng.uniform(1, 6, n)], 6, 9, 4.0,
                     list(10.0 ** rng.uniform(-4, -2, n)), list(10.0 ** rng.uniform(-3, -1, n)),
                     list(rng.uniform(0, 1, n)), formal_solver=fs)
    _check(p)


@pytest.mark.parametrize("rays", RAYS, ids=lambda r: f"{r[0]}x{r[1]}")
def test_ray_layouts(rays):
    m, nc = rays
    p = W.make_slabs([70, 20], [(1e-3, 1e4), (1e-2, 1e2)], 2 * m, nc, 4.0, [1e-3, 5e-3],
                     [1e-2, 1e-1], [0.5, 0.9])
    # no two opacities equal, so every frequency keeps its ray
    _check(p.with_(opac=p.opac * np.exp(0.02 * p.x)[None, :]))
