"""The sources beside the package are the ones its build compiles or includes: no second copy of a kernel that would go its own way."""
import os

from paper_2507_12205_amd import build


def test_every_source_is_built():
    used = {os.path.normpath(os.path.join(build.CSRC, f)) for f in build.SOURCES + build.HEADERS}
    assert {os.path.join(build.CSRC, f) for f in os.listdir(build.CSRC)} == {f for f in used if os.path.dirname(f) == build.CSRC}
