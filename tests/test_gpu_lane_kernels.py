"""Widths whose scatter or gather is not the matrix kernel.

The tile kernels are chosen by precision and widths: in FP32 the scatter of W = 1
and 2 and of W_z = 1, in FP64 that of (7, 1), take lanes that own residues; the
gather takes lanes that own records in FP32, and in FP64 up to W = 5.  One pair on
each side of every line, with the clumps of test_gpu_windows.py: plain calls,
whose records are ordered for their own direction, and shared-binning calls,
whose records are ordered for both, against the FP64 oracle.
"""
import pytest

import test_gpu_windows as windows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,Wz", [(1, 1), (3, 3), (4, 4), (6, 6), (3, 1), (5, 1), (6, 1), (7, 1), (7, 2), (8, 1)])
def test_clumps_beside_the_rule(W, Wz):
    windows.test_clumps(W, Wz)
