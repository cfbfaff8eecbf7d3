"""bf16 products whose sizes end inside a tile, a slab or a weight part.

B T no multiple of the 64-deep slab (the weight gradients' K), a width that
is an odd multiple of 64 (Q, K, V columns then end inside a column tile), a
batch of one chunked call (the carried memory's products have B rows), and
small products on 32-row tiles with a last tile of one row.  Bounds as in
test_gpu_parity.
"""

import pytest

from test_gpu_parity import compare, inputs, run_gpu, run_oracle, say, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,D,H,L", [
    (1, 65, 192, 3, 16),     # 65 rows, 192 = 1.5 column tiles per part
    (2, 1033, 320, 5, 128),  # 2066 rows, K ends 18 into a slab
    (9, 1027, 192, 3, 64),   # 9243 rows: 128-row tiles and partial parts
    (3, 7, 64, 1, 4),        # 21 rows, one half-empty column tile
])
def test_tails(torch_cuda, B, T, D, H, L):  # noqa: F811
    say(f"case B={B} T={T} D={D} L={L}")
    X, W, dY = inputs(B, T, D, "bf16", w_std=0.05)
    gpu = run_gpu(torch_cuda, B, T, D, H, L, "bf16", X, W, dY)
    compare(gpu, run_oracle(B, T, D, H, L, X, W, dY), "bf16", f"tails-{B}x{T}x{D}")
