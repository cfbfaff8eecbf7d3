"""Decoding products at the edges of their tiles (128 columns, 16 sequences,
128 rows a workgroup): widths with half a column tile and a partial last
workgroup of rows, batches of one, of a full tile, of one more and of several.
Bounds as in test_gpu_decode.
"""

import numpy as np
import pytest

from conftest import maxabs_rel
from test_gpu_decode import gpu_decode, oracle_y
from test_gpu_parity import inputs, say, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,D", [(1, 64), (16, 192), (17, 320), (40, 128), (64, 448)])
def test_decode_tiles(torch_cuda, B, D):  # noqa: F811
    T, L, H = 21, 9, D // 64  # two block ends
    say(f"decode B={B} D={D}")
    X, W, _ = inputs(B, T, D, "bf16", w_std=0.05)
    got = gpu_decode(torch_cuda, B, T, D, H, L, "bf16", X, W, 0.8, True)
    ref = oracle_y(B, T, D, H, L, X, W, 0.8, True)
    assert np.isfinite(got).all()
    assert maxabs_rel(got, ref) <= 2e-2
