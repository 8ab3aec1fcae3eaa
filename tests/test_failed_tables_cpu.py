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


GROUPS = """
ns = [40, 70, 33, 200, 17, 90]
p = W.make_slabs(ns, [(1e-3, 1e4)] * 6, 8, 21, 5.0, [1e-3] * 6, [1e-2] * 6, [0.5] * 6)
p = p.with_(opac=p.opac * (1 + 1e-3 * np.arange(21)))  # as many rays as frequencies
A = (ctypes.c_double * 16)()
go = lambda h: B._check(B.lib().rt_assemble(h._h, (ctypes.addressof(A) + 15) // 16 * 16, None))
with B.setup(p) as h:
    rt.host_largest()
    first, again = launches(lambda: go(h)), launches(lambda: go(h))
    tables = rt.host_largest()
    # the (E, w) of every interval and ray is what the assembly cannot do without
    assert tables > 16 * sum(n - 1 for n in ns) * 4 * 21
for limit, groups in ((tables - 1, 2), (tables * 200 // 450, 0)):
    with B.setup(p) as h:
        rt.host_limit(max(limit, 16 * sum(n - 1 for n in ns) * 4 * 21))
        n1, n2 = launches(lambda: go(h)), launches(lambda: go(h))
        # in every call, a table and an assembly for each group
        assert n2 >= again + 2 * 2 - 1 and n1 == n2 + 1
        if groups:
            assert n2 == again + 2 * groups - 1
    rt.host_limit(0)
with B.setup(p) as h:
    rt.host_limit(1000)  # no room at all
    assert fails(lambda: go(h)) == B.RT_ENOMEM
    rt.host_limit(0)
    assert launches(lambda: go(h)) == first
assert rt.host_live() == 0
"""


def test_assembly_in_groups_where_the_tables_do_not_fit(so):
    """A limit on an allocation that the (E, w) table meets and the tables of
    all slabs do not: the assembly runs in groups of slabs."""
    HL.run(so, GROUPS)
