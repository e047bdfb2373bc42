"""Registers and scratch of the built kernels (code object metadata, no GPU)."""
import os
import re

import pytest

from paper_2608_02134_amd import binding as B

from .code_objects import kernels


@pytest.fixture(scope="module")
def built():
    if not os.path.exists(B.LIB_PATH):
        pytest.fail("libgmc.so is not built; run __graft_entry__.build()")
    return kernels(B.LIB_PATH)


def _find(built, pattern):
    found = {n: k for n, k in built.items() if re.search(pattern, n)}
    assert found, pattern
    return found


def test_head_gram_keeps_its_registers(built):
    """No probe rank (1..8, with and without 16-byte runs) spills to scratch."""
    found = _find(built, r"headgram_kernelILi\dELb[01]")
    assert len(found) == 16
    assert {n: k[".private_segment_fixed_size"] for n, k in found.items() if k[".private_segment_fixed_size"]} == {}
