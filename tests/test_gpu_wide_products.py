"""The 256 x 256 product kernel at the edges of its tiles.

Large bf16 products run on 256 x 256 tiles where a time model of the two
kernels says so; which products of a case do is asserted, so that a change of
the model cannot move a case off the kernel unseen.  The last row tiles have
64 to 127 rows, the last column tiles 128 columns; with 1920 columns every
epilogue of the layer meets both.  Sampled sequences, the last (in the last
row tile) among them, are compared with the float64 oracle as in
test_gpu_full_size.  Bound: 2e-2; the rounding model of bf16 storage
(bf16_model.py, 12 realisations) errs by at most 5.7e-3 on any case, the decay
gradient by 3.3e-3, with 1920 columns by 2.4e-3 (and other outputs by 5.9e-3).

And the language model's products: its MLP's with d = 576 over 14104 rows (a
last row tile of 24, a last column tile of 64), its head's with d = 768 over
2000 rows and 7492 words (7552 padded columns, 29.5 tiles).  Bounds as in
test_gpu_model; the rounding model (lm_bf16_model.py) errs by at most 8.4e-3
and 1.02e-2.
"""

import numpy as np
import pytest

from test_gpu_full_size import sampled_case, torch_cuda  # noqa: F401
from test_gpu_model import GRAD_TOL, LOSS_TOL, oracle_params
from test_gpu_parity import say
from test_product_plans import WIDE, layer_plans, model_plans

pytestmark = pytest.mark.gpu

ALL = {"qkv", "score", "gate", "hbar", "dgrad", "dx"}


@pytest.mark.parametrize("B,T,D,H,L,rows,residual,wide", [
    (129, 255, 1152, 18, 60, [0, 128], False, {"qkv", "dx"}),
    (16, 1028, 1024, 16, 128, [15], False, {"qkv"}),
    (4, 1561, 1920, 30, 128, [0, 3], True, ALL),
    (4, 1817, 1920, 30, 128, [1, 3], False, ALL),
])
def test_wide_tile_edges(torch_cuda, B, T, D, H, L, rows, residual, wide):  # noqa: F811
    plans = layer_plans(B, T, D, "bf16", residual)
    assert {k for k in ALL if plans[k][0] == WIDE} == wide
    sampled_case(torch_cuda, f"wide-{B}x{T}x{D}", B, T, D, H, L, rows=rows, P=T,
                 residual=residual)


@pytest.mark.parametrize("V,d,H,B,T,wide", [
    (836, 576, 9, 4, 3526, {"mlp_out"}),
    (7492, 768, 12, 2, 1000, {"stats", "grad"}),
])
def test_wide_model_products(torch_cuda, V, d, H, B, T, wide):  # noqa: F811
    from oracle import model_oracle as mo
    from paper_2608_13578_amd.inputs import make_model_inputs
    from paper_2608_13578_amd.model import ModelBuffers
    nl, L = 1, 128
    assert {k for k, v in model_plans(V, d, B, T).items() if v[0] == WIDE} == wide
    say(f"model V={V} d={d} B={B} T={T}")
    torch = torch_cuda
    arrs, tok, tgt = make_model_inputs(V, d, T, nl, B, w_std=0.03)
    mb = ModelBuffers(V, d, H, nl, B, T, L, 0.8)
    mb.set_params(arrs)
    mb.step(torch.from_numpy(tok).cuda(), torch.from_numpy(tgt).cuda())
    torch.cuda.synchronize()
    say("GPU step done")
    loss, cache = mo.forward(tok.astype(np.int64), tgt.astype(np.int64), oracle_params(arrs, nl),
                             L, H, 0.8)
    G = mo.flatten(mo.backward(cache))
    assert abs(float(mb.loss.item()) - loss) <= LOSS_TOL
    for name, g, r in zip(mb.names, mb.arrays(mb.grads), G):
        g, r = np.asarray(g).reshape(-1), np.asarray(r).reshape(-1)
        err = float(np.abs(g - r).max() / max(np.abs(r).max(), 1e-30))
        assert err <= GRAD_TOL, (name, err)
