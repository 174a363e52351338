"""Launch shapes, which the host computes for every call: a small program over the
library's internal header prints them (no GPU call is made here)."""
import os
import shutil
import subprocess

import pytest

from paper_2111_02912_amd import _lib, build


def test_launches_compute_no_splits():
    """The column passes' thread counts are constants of their kernels, not
    searched for again at every launch."""
    if not shutil.which("nm"):
        pytest.skip("no nm")
    names = subprocess.run(["nm", "-C", _lib.LIB_PATH], capture_output=True, text=True, check=True).stdout
    assert "k_any_cols" in names
    for f in ("col_threads(", "row_lines(", "split_cost(", "split_radices("):
        assert f not in names, f
