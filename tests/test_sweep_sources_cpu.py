"""The hash that stored launch plans and counter readings are trusted by covers
what decides a sweep's speed: the kernels and also the code that lays out its
rays and blocks, with the declarations they share."""
import glob
import os
import re
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

from paper_2110_11873_amd.csrc import build  # noqa: E402


def test_sources_that_lay_out_or_sweep_blocks_are_hashed():
    plans = re.compile(r"BlockDesc [a-z_]+\{\}|struct (BlockDesc|AtmDesc|SweepArgs) \{|chunk_len\(int|merge_frequencies\(const"
                       r"|sweep_kernel\(SweepArgs|finalize_point\(const")
    found = {os.path.basename(f) for f in glob.glob(os.path.join(build.HERE, "*.h*")) if plans.search(open(f).read())}
    assert len(found) >= 5 and found <= set(build.SWEEP_SOURCES), found - set(build.SWEEP_SOURCES)


def test_every_sweep_source_is_built_or_included():
    for f in build.SWEEP_SOURCES:
        assert f.endswith(".h") or f in build.SOURCES, f
