"""A table whose launch or wait failed is made again by the next call: the second
call launches as much as a first one, and nothing is left allocated at the end."""
import pytest

from tests import host_library as HL


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    return HL.build(tmp_path_factory.mktemp("runtime"))


REDISTRIBUTION = """
p = W.make_slabs([40], [(1e-3, 1e4)], 8, 21, 5.0, [1e-3], [1e-2], [0.5])
R = W.redistribution_matrix(p.x, p.w_nu, p.phi[0], 0.5)
with B.setup(p) as h:
    first = launches(lambda: h.set_redistribution(R))
    assert first == 1
with B.setup(p) as h:
    {fail}
    assert fails(lambda: h.set_redistribution(R)) == B.RT_EDEVICE
    assert launches(lambda: h.set_redistribution(R)) == first
    assert launches(lambda: h.set_redistribution(R)) == 0
assert rt.host_live() == 0
"""


@pytest.mark.parametrize("fail", ["rt.host_fail_launch(1)", "rt.host_fail_sync(1)"])
def test_redistribution_table(so, fail):
    HL.run(so, REDISTRIBUTION.format(fail=fail))


ASSEMBLY = """
p = W.make_slabs([40, 70], [(1e-3, 1e4)] * 2, 8, 21, 5.0, [1e-3] * 2, [1e-2] * 2, [0.5] * 2)
A = (ctypes.c_double * 16)()
go = lambda h: B._check(B.lib().rt_assemble(h._h, (ctypes.addressof(A) + 15) // 16 * 16, None))
with B.setup(p) as h:
    first, again = launches(lambda: go(h)), launches(lambda: go(h))
    assert first > again > 0
with B.setup(p) as h:
    rt.host_fail_launch({n})
    assert fails(lambda: go(h)) == B.RT_EDEVICE
    assert launches(lambda: go(h)) == first
    assert launches(lambda: go(h)) == again
assert rt.host_live() == 0
"""


@pytest.mark.parametrize("n", [1, 2])
def test_assembly_tables(so, n):
    HL.run(so, ASSEMBLY.format(n=n))
