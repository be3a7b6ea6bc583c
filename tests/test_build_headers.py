"""An incremental build compiles the sources again after a change to any header.  No GPU, no compiler needed."""
import glob
import os

import pytest

from paper_2411_15871_amd import build as B

HEADERS = sorted(glob.glob(os.path.join(B.CSRC, "*.h")) + [os.path.join(B.HERE, "..", "include", "dhelix.h")])


@pytest.mark.parametrize("header", HEADERS, ids=os.path.basename)
def test_every_header_counts(header, monkeypatch):
    real = os.path.getmtime
    monkeypatch.setattr(B.os.path, "getmtime", lambda p: 4e9 if os.path.realpath(p) == os.path.realpath(header) else real(p))
    assert B._deps_mtime() == 4e9
