"""Edges of the tiles, panels and splits that the kernels cut their work into, against the fp64 oracle.

The bounds are harness.check's: the parity bound of the types and, with fp32 records, the regression guard.
"""
import numpy as np
import pytest

import harness as H
from test_gpu_parity import _direct_case, say

pytestmark = pytest.mark.gpu

TYPES = [("bf16", "f32"), ("f16", "f32"), ("bf16", "bf16"), ("f16", "f16")]


@pytest.mark.parametrize("in_dtype, rec_dtype", TYPES)
@pytest.mark.parametrize("block_size", [None, 16])
def test_direct_second_panel(in_dtype, rec_dtype, block_size):
    """Contexts around the end of the first 64-row panel and around every 16-row block of the second."""
    lens = np.array([0, 1, 63, 64, 65, 66, 79, 80, 81, 95, 97, 112, 113, 127, 128], np.int32)
    e = _direct_case(B=len(lens), Hk=2, Hv=4, d=128, Lmax=128, cap=128, in_dtype=in_dtype, seed=800, lens=lens,
                     then_decode=False, rec_dtype=rec_dtype, out_dtype=rec_dtype, block_size=block_size)
    say("direct, second panel, %s/%s: rel err out/u/decode/state %.2e %.2e %.2e %.2e" % ((in_dtype, rec_dtype) + e))
    H.check(e, in_dtype, rec_dtype, "second panel")
