"""Compile-time twiddle factors against long-double cosines and sines (host
compiler, no GPU)."""
import shutil

import pytest

from tests.test_arena import SANITIZE, _run_native


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
@pytest.mark.parametrize("sanitize", [False, True])
def test_unit_roots_correctly_rounded(sanitize):
    _run_native("unit_root_check.cpp", SANITIZE if sanitize else [], "unit_root" + ("_san" if sanitize else ""))
