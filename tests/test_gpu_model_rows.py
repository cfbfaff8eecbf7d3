"""The model's row kernels at the edges of their ranges.

LayerNorm widths on each of its kernels (64 and 128 columns forward and
backward, 512 backward only, 192 on neither vector form), rows that end
inside every workgroup's share, and a batch where half of the tokens are one
id and the rest repeat, as text does (the lookup gradient groups them).
Bounds as in test_gpu_model.  And the weight gradients on the second stream
against one stream: the same bits, apart from the atomics of E's gradient.
"""

import numpy as np
import pytest

from test_gpu_model import GRAD_TOL, LOSS_TOL, oracle_params
from test_gpu_parity import say, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu


def step(torch, V, d, H, nl, B, T, L, tok, tgt, arrs, side):
    from paper_2608_13578_amd.model import ModelBuffers
    mb = ModelBuffers(V, d, H, nl, B, T, L, 0.8, side=side)
    mb.set_params(arrs)
    mb.step(torch.from_numpy(tok).cuda(), torch.from_numpy(tgt).cuda())
    torch.cuda.synchronize()
    return mb


@pytest.mark.parametrize("d,H,w_std", [(64, 4, 0.1), (128, 8, 0.1), (192, 3, 0.05), (512, 8, 0.03)])
def test_rows(torch_cuda, d, H, w_std):  # noqa: F811
    from oracle import model_oracle as mo
    from paper_2608_13578_amd.inputs import make_model_inputs
    V, nl, B, T, L = 60, 1, 3, 101, 32  # 303 rows
    say(f"model rows d={d}")
    arrs, tok, tgt = make_model_inputs(V, d, T, nl, B, w_std=w_std)
    tok[np.random.default_rng(3).random(tok.shape) < 0.5] = 7
    mb = step(torch_cuda, V, d, H, nl, B, T, L, tok, tgt, arrs, True)
    loss, cache = mo.forward(tok.astype(np.int64), tgt.astype(np.int64), oracle_params(arrs, nl), L,
                             H, 0.8)
    G = mo.flatten(mo.backward(cache))
    assert abs(float(mb.loss.item()) - loss) <= LOSS_TOL
    for name, g, r in zip(mb.names, mb.arrays(mb.grads), G):
        g, r = np.asarray(g).reshape(-1), np.asarray(r).reshape(-1)
        err = float(np.abs(g - r).max() / max(np.abs(r).max(), 1e-30))
        assert err <= GRAD_TOL, (name, err)


def test_second_stream_changes_nothing(torch_cuda):  # noqa: F811
    from paper_2608_13578_amd.inputs import make_model_inputs
    V, d, H, nl, B, T, L = 97, 128, 8, 3, 4, 512, 64
    arrs, tok, tgt = make_model_inputs(V, d, T, nl, B)
    a, b = (step(torch_cuda, V, d, H, nl, B, T, L, tok, tgt, arrs, side) for side in (True, None))
    for name, x, y in zip(a.names, a.arrays(a.grads), b.arrays(b.grads)):
        if name == "E":  # lookups add with float32 atomics, in any order
            assert np.abs(x - y).max() <= 1e-5 * np.abs(y).max()
        else:
            assert np.array_equal(x, y), name
