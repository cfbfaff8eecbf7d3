"""The 256 x 256 product kernel at the edges of its tiles.

Large bf16 products run on 256 x 256 tiles where a time model of the two
kernels says so.  These layers reach it with a last row tile of 127 and of 64
rows and a last column tile of 128, next to epilogues of every kind; sampled
sequences, the last (in the last row tile) among them, are compared with the
float64 oracle as in test_gpu_full_size.  Bound: 2e-2; the rounding model of
bf16 storage (bf16_model.py, 12 realisations) errs by at most 5.7e-3 on
either case, the decay gradient by 3.3e-3.
"""

import pytest

from test_gpu_full_size import sampled_case, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,D,H,L,rows", [
    (129, 255, 1152, 18, 60, [0, 128]),  # 32895 rows, 1152 columns (4.5 tiles)
    (16, 1028, 1024, 16, 128, [15]),     # 16448 rows: 64 whole tiles and 64 rows
])
def test_wide_tile_edges(torch_cuda, B, T, D, H, L, rows):  # noqa: F811
    sampled_case(torch_cuda, f"wide-{B}x{T}x{D}", B, T, D, H, L, rows=rows, P=T)
