"""The backward passes' second stream: used from a certain size on, and then
with the same bits as on one stream.

Layers just past the sizes from which their weight gradients fork, of every
kind of backward that forks (whole, chunked with accumulation, one decay per
channel, float32; the narrow layer by B T D, the others by B T D^2), one just
below, and models on both sides.  Whether a pass used the second stream is
seen from a kernel that keeps that stream busy: a pass that forked joins it,
so its own stream ends after that kernel.
"""

import numpy as np
import pytest

from test_gpu_parity import inputs, say, torch_cuda  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [
    # B, T, D, H, L, dtype, channel, chunks, forks
    (2, 4608, 384, 6, 128, "bf16", False, 1, True),   # B T D^2 = 1.36e9
    (2, 1088, 768, 12, 100, "bf16", True, 1, True),   # 1.28e9
    (2, 4608, 384, 6, 128, "bf16", False, 2, False),  # 0.68e9 a chunk
    (2, 4352, 768, 12, 128, "bf16", False, 4, True),  # 1.28e9 a chunk
    (8, 12288, 64, 4, 64, "bf16", False, 1, True),    # B T D = 6.3e6
    (1, 1024, 384, 6, 64, "f32", False, 1, True),     # 1.5e8
    (1, 1024, 320, 5, 64, "f32", False, 1, False),    # 1.05e8
]


def layers(case, side):
    from paper_2608_13578_amd.layer import LayerBuffers
    B, T, D, H, L, dtype, channel, chunks, _ = case
    gamma = np.linspace(0.6, 0.9, D).astype(np.float32) if channel else 0.8
    n = T // chunks
    return [LayerBuffers(B, n, D, H, L, gamma=gamma, dtype=dtype, side=side,
                         accumulate=k + 1 < chunks) for k in range(chunks)]


def run(torch, case, side, busy=None):
    """(outputs, whether the pass's stream ended after `busy` did)"""
    from paper_2608_13578_amd.layer import to_device
    B, T, D, H, L, dtype, channel, chunks, _ = case
    X, W, dY = inputs(B, T, D, dtype, w_std=0.05)
    lbs = layers(case, side)
    n = T // chunks
    part = [slice(k * n, (k + 1) * n) for k in range(chunks)]
    Xs = [to_device(np.ascontiguousarray(X[:, p]), dtype) for p in part]
    dYs = [to_device(np.ascontiguousarray(dY[:, p]), dtype) for p in part]
    Ys, dXs = [lb.new_activation() for lb in lbs], [lb.new_activation() for lb in lbs]
    for lb in lbs:
        lb.set_params(W)
    g = lbs[0].new_grads()
    after = None
    # twice: the first pass loads the kernels
    for again in range(2):
        for t in g.values():
            t.zero_()
        carries = [lb.new_carry() for lb in lbs]
        dcarries = [lb.new_carry() for lb in lbs]
        if chunks == 1:
            lbs[0].forward(Xs[0], Ys[0])
        else:
            for k, lb in enumerate(lbs):
                lb.forward_chunk(Xs[k], Ys[k], carries[k - 1] if k else None, carries[k])
        torch.cuda.synchronize()
        if busy is not None and again:
            done = busy()
        if chunks == 1:
            lbs[0].backward(Xs[0], dYs[0], dXs[0], g)
        else:
            for k in reversed(range(chunks)):
                lbs[k].backward_chunk(Xs[k], dYs[k], dcarries[k + 1] if k + 1 < chunks else None,
                                      dXs[k], dcarries[k], g)
        torch.cuda.current_stream().synchronize()
        if busy is not None and again:
            after = done.query()
        torch.cuda.synchronize()
    return {"Y": torch.cat(Ys, 1), "dX": torch.cat(dXs, 1), **g}, after


def occupy(torch, side):
    """A kernel of tens of milliseconds or more on the second stream, and the
    event at its end."""
    def start():
        done = torch.cuda.Event()
        with torch.cuda.stream(side.stream):
            torch.cuda._sleep(100_000_000)
            done.record()
        assert not done.query()
        return done
    return start


@pytest.fixture(scope="module")
def side(torch_cuda):  # noqa: F811
    """A second stream that does not share its hardware queue with the tests'
    own stream (streams are dealt to a few queues; on a shared one everything
    waits for the occupying kernel)."""
    from paper_2608_13578_amd.layer import SideStream
    torch = torch_cuda
    x = torch.zeros(64, device="cuda")
    for _ in range(8):
        s = SideStream()
        done = occupy(torch, s)()
        x.add_(1.0)
        torch.cuda.current_stream().synchronize()
        apart = not done.query()
        torch.cuda.synchronize()
        if apart:
            return s
    pytest.skip("every second stream shares the hardware queue of the first")


@pytest.mark.parametrize("case", CASES)
def test_layer(torch_cuda, side, case):  # noqa: F811
    say(f"case {case}")
    two, used = run(torch_cuda, case, side, occupy(torch_cuda, side))
    one, _ = run(torch_cuda, case, None)
    assert used == case[-1]
    for k, v in one.items():
        assert torch_cuda.equal(two[k], v), k


@pytest.mark.parametrize("V,d,B,T,forks", [
    (10000, 256, 8, 512, True),   # B T d^2 = 2.7e8, the head's B T V d 1.05e10
    (1000, 256, 8, 512, False),   # 1.05e9
    (1000, 512, 4, 1024, True),   # B T d^2 = 1.07e9
    (97, 128, 4, 512, False),
])
def test_model(torch_cuda, side, V, d, B, T, forks):  # noqa: F811
    from paper_2608_13578_amd.inputs import make_model_inputs
    from paper_2608_13578_amd.model import ModelBuffers
    torch = torch_cuda
    say(f"model V={V} d={d} B={B} T={T}")
    arrs, tok, tgt = make_model_inputs(V, d, T, 2, B)
    tok, tgt = torch.from_numpy(tok).cuda(), torch.from_numpy(tgt).cuda()
    grads = []
    for second in (side, None):
        mb = ModelBuffers(V, d, d // 64, 2, B, T, 64, 0.8, side=second)
        mb.set_params(arrs)
        mb.step(tok, tgt)
        torch.cuda.synchronize()
        if second:
            done = occupy(torch, second)()
            mb.step(tok, tgt)
            torch.cuda.current_stream().synchronize()
            assert done.query() == forks
            torch.cuda.synchronize()
        grads.append((mb, mb.arrays(mb.grads)))
    (mb, a), (_, b) = grads
    for name, x, y in zip(mb.names, a, b):
        if name == "E":  # lookups add with float32 atomics, in any order
            assert np.abs(x - y).max() <= 1e-5 * np.abs(y).max()
        else:
            assert np.array_equal(x, y), name
