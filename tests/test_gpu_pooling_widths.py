"""Whole-row pooling at widths whose vectors do not divide into full waves.

From 192 blocks on, pooling runs one workgroup per block with whole rows per
thread group; at these widths the threads of a row are no divisor of 512, so
the last wave is partly idle.  Bounds as in test_gpu_parity.
"""

import pytest

from test_gpu_parity import compare, inputs, run_gpu, run_oracle, say, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,dtype", [(576, "bf16"), (1152, "bf16"), (704, "f32"), (1984, "f32")])
def test_many_blocks(torch_cuda, D, dtype):  # noqa: F811
    B, T, H, L = 2, 99 * 8 + 3, D // 64, 8  # 100 blocks a sequence, the last of 3 tokens
    say(f"case D={D} {dtype}")
    X, W, _ = inputs(B, T, D, dtype)
    gpu = run_gpu(torch_cuda, B, T, D, H, L, dtype, X, W)
    compare(gpu, run_oracle(B, T, D, H, L, X, W), dtype, f"pool-{D}-{dtype}")
