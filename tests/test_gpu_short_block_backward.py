"""The fused attention backward of blocks of at most 32 tokens, right after
a launch that left NaN in the same place of the LDS.

Such a block fills half of its 64-row tile; the other half's row sums
(delta) take part multiplied by zero probabilities, so they must be finite
whatever the LDS held.
"""

import numpy as np
import pytest

from test_gpu_parity import compare, inputs, run_gpu, run_oracle, say, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [20, 32])
def test_short_blocks_after_nan(torch_cuda, L):  # noqa: F811
    B, T, D, H = 3, 98, 256, 4
    X, W, dY = inputs(B, T, D, "bf16")
    ref = run_oracle(B, T, D, H, L, X, W, dY)
    # 16 times the blocks of 64 tokens (the same LDS layout), upstream NaN
    say(f"case L={L}: a backward of NaN, then the layer")
    Xb, Wb, dYb = inputs(64, 256, D, "bf16")
    run_gpu(torch_cuda, 64, 256, D, H, 64, "bf16", Xb, Wb, np.full_like(dYb, np.nan))
    compare(run_gpu(torch_cuda, B, T, D, H, L, "bf16", X, W, dY), ref, "bf16", f"short-L{L}")
