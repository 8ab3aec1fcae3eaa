"""A stored launch plan belongs to a number of distinct opacities, on which the
rays of the sweep and so its plan depend: the key separates problems of one shape
by it.  Even profiles, for which the shipped plans are measured, keep their key."""
import os
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

from paper_2110_11873_amd import autotune as AT  # noqa: E402
from paper_2110_11873_amd import workloads as W  # noqa: E402


def key(p):
    return AT.shape_key(p, False, "gfx950")


@pytest.mark.parametrize("make", [W.config2, lambda: W.config4(20), lambda: W.make_slabs([30] * 3, [(1e-3, 1e4)] * 3, 4, 10, 5.0, [1e-3] * 3, [1e-2] * 3, [0.5] * 3)])
def test_key_separates_numbers_of_distinct_opacities(make):
    p = make()
    f = 1 + 1e-3 * np.arange(p.n_nu)
    shifted = p.with_(opac=p.opac * f)
    one = p.with_(opac=np.vstack([p.opac[:-1], p.opac[-1:] * f]))  # the largest count of the slabs counts
    half = p.with_(opac=p.opac * np.where(np.arange(p.n_nu) < 3, 1.001, 1.0))
    assert len({key(p), key(shifted), key(half)}) == 3
    assert key(one) == key(shifted)
    assert key(p.with_(opac=p.opac * (1 + 1e-15 * np.arange(p.n_nu)))) == key(p)
    # all that follows from the shape alone is the same
    assert key(p).split("|")[:-1] == key(shifted).split("|")[:-1]


def test_even_profiles_keep_the_key_of_the_shipped_plans():
    keys = {ln.split()[0] for ln in open(AT.index_path(AT.DEFAULT_CACHE)) if ln.strip() and not ln.startswith("#")}
    for p in (W.config2(), W.config3(), W.config4(512)):
        assert key(p) in keys


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_a_problem_that_is_not_one_has_the_key_of_its_shape(bad):
    p = W.config2()
    opac = p.opac.copy()
    opac[0, 5:9] = bad
    assert key(p.with_(opac=opac)) == key(p)
