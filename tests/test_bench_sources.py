"""bench.py drops a recorded conv profile when a source that conv and dense
calls are built from changes: its list holds all of them."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402
from paper_1810_11066_amd import build  # noqa: E402


def test_conv_sources_are_what_the_library_is_built_from():
    listed = [os.path.basename(f) for f in bench.CONV_SOURCES]
    assert len(listed) == len(set(listed))
    # the entry points and the pack kernels launch no conv kernel of their own
    assert set(listed) == set(build.SOURCES) - {"api.hip", "quant_pack.hip"}
