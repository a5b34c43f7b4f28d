"""Registers of kernels whose speed rests on the wavefronts that fit a SIMD,
from the built library's own metadata."""
import os

import pytest

from kernel_resources import find, kernels, wavefronts
from paper_1608_04118_amd import binding as B


@pytest.fixture(scope="module")
def table():
    if not os.path.exists(B.LIB_PATH):
        from paper_1608_04118_amd import build
        build.build()
    return kernels(B.LIB_PATH)


# one sweep of the adjoint: step, seed, initialisation (adjoint storage, arithmetic, fields)
@pytest.mark.parametrize("types,least", [("fff", (5, 8, 6)), ("ffd", (4, 8, 5)), ("ddd", (2, 4, 3))],
                         ids=["f32", "f32sr", "f64"])
def test_single_adjoint_sweep(table, types, least):
    for mode, waves in enumerate(least):
        assert wavefronts(find(table, "adjoint_kernel", "%sLi%dE" % (types, mode))) >= waves, (types, mode)
