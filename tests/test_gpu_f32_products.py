"""Float32 products at the edges of their tiles.

64 x 64 tiles where they give every CU a workgroup, 32 x 64 below that; the
last row tile, the last column tile (D = 320) and the last 32-deep slab of
the weight gradients (K = B T) are partial.  Bounds as in test_gpu_parity.
"""

import pytest

from test_gpu_parity import compare, inputs, run_gpu, run_oracle, say, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,D,H,L", [
    (2, 2063, 320, 5, 50),  # 4126 rows: 64-row tiles, 30 rows in the last
    (1, 65, 320, 5, 16),    # 65 rows: 32-row tiles, one row in the last
    (3, 11, 64, 1, 4),      # 33 rows, one column tile
])
def test_f32_tile_edges(torch_cuda, B, T, D, H, L):  # noqa: F811
    say(f"case B={B} T={T} D={D} L={L}")
    X, W, dY = inputs(B, T, D, "f32", w_std=0.05)
    gpu = run_gpu(torch_cuda, B, T, D, H, L, "f32", X, W, dY)
    compare(gpu, run_oracle(B, T, D, H, L, X, W, dY), "f32", f"f32-edges-{B}x{T}x{D}")
