"""Float32 products at the edges of their tiles.

64 x 64 tiles where they give every CU a workgroup, 32 x 64 below that; the
last row tile, the last column tile (D = 320) and the last 32-deep slab of
the weight gradients (K = B T) are partial.  And more rows than 65535 tiles of
64, which the grid's second and third dimensions could not hold.  Bounds as in
test_gpu_parity.
"""

import numpy as np
import pytest

from test_gpu_parity import GRADS, compare, inputs, run_gpu, run_oracle, say, torch_cuda  # noqa: F401

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


def test_more_rows_than_65535_tiles(torch_cuda):  # noqa: F811
    """1024 sequences of 4097 tokens, D = 64: 65553 tiles of 64 rows.  The first
    and the last sequence are compared whole; the upstream gradient is zero on
    the others, so the weight gradients are those two sequences' alone."""
    from paper_2608_13578_amd.layer import LayerBuffers, to_device, to_host64
    torch, rows = torch_cuda, [0, 1023]
    B, T, D, H, L = 1024, 4097, 64, 1, 128
    assert B * T > 65535 * 64
    say(f"case B={B} T={T} D={D}")
    X, W, dY = inputs(2, T, D, "f32", w_std=0.05)
    lb = LayerBuffers(B, T, D, H, L, dtype="f32")
    lb.set_params(W)
    Xd = torch.randn((B, T, D), generator=torch.Generator("cuda").manual_seed(3), device="cuda")
    dYd = torch.zeros((B, T, D), device="cuda")
    Xd[rows], dYd[rows] = to_device(X, "f32"), to_device(dY, "f32")
    Yd, dXd, g = lb.new_activation(), lb.new_activation(), lb.new_grads()
    lb.forward(Xd, Yd)
    lb.backward(Xd, dYd, dXd, g)
    torch.cuda.synchronize()
    assert not bool(dXd[1:-1].any())
    gpu = {"Y": to_host64(Yd[rows]), "dX": to_host64(dXd[rows]),
           "dgamma": float(g["dgamma"][0].item()), **{k: to_host64(g[k]) for k in GRADS}}
    assert all(np.isfinite(v).all() for v in gpu.values())
    compare(gpu, run_oracle(2, T, D, H, L, X, W, dY), "f32", "f32-many-rows")
