"""How the library deals its matrix products to kernels and grids, on the CPU.

The library reports the plan of a product (bcmt_internal_product_plan: the
function that launches them takes the same one).  Every product of the
largest accepted layers must have a grid within the limits of a launch: 2^31 -
1 in x, 65535 in y and z.
"""

import ctypes
import os

import pytest

# kernels (ProductKernel) and epilogues (EpiKind) of csrc/gemm.hip
F32_32, F32_64, PIPE_32, PIPE_8, PIPE_4, WIDE = range(6)
STORE, SCORE, GATE, HBAR, GELU, GELU_BWD, HEAD_STATS, HEAD_GRAD, PARTIAL, STORE_ADD, GATE_X = range(11)
SEG_N, SEG_K = 1, 2


def plan(dtype, kind, M, N, K, amc=False, bnc=True, seg=0, seg_len=0, min_k=0):
    """(kernel, (grid x, y, z), K range of a split)"""
    from paper_2608_13578_amd import bcmt as abi
    out = (ctypes.c_int * 5)()
    abi.lib().bcmt_internal_product_plan(int(dtype == "bf16"), kind, M, N, K, int(amc), int(bnc),
                                         seg, seg_len, min_k, out)
    return out[0], tuple(out[1:4]), out[4]


def layer_plans(B, T, D, dtype, residual=False):
    """The products of a layer's forward and backward over B T rows."""
    BT = B * T
    p = {"qkv": plan(dtype, STORE, BT, 3 * D, D, seg=SEG_N, seg_len=D),
         "score": plan(dtype, SCORE, BT, D, D),
         "gate": plan(dtype, GATE_X if residual else GATE, BT, D, D),
         "hbar": plan(dtype, HBAR, BT, D, D, bnc=False),
         "dgrad": plan(dtype, STORE, BT, D, D, bnc=False),
         "dx": plan(dtype, STORE_ADD if residual else STORE, BT, D, 3 * D, bnc=False, seg=SEG_K, seg_len=D),
         "dWqkv": plan(dtype, PARTIAL, D, 3 * D, BT, amc=True, min_k=128),
         "dWm": plan(dtype, PARTIAL, D, D, B, amc=True, min_k=512)}
    for mk in (128, 256, 512):
        p[f"dW-{mk}"] = plan(dtype, PARTIAL, D, D, BT, amc=True, min_k=mk)
    return p


def model_plans(V, d, B, T):
    """The MLP and head products of a language model's step (its layers: layer_plans)."""
    BT, Vp = B * T, (V + 127) // 128 * 128
    return {"gelu": plan("bf16", GELU, BT, 4 * d, d),
            "gelu_bwd": plan("bf16", GELU_BWD, BT, 4 * d, d, bnc=False),
            "mlp_out": plan("bf16", STORE_ADD, BT, d, 4 * d),
            "stats": plan("bf16", HEAD_STATS, BT, Vp, d, bnc=False),
            "grad": plan("bf16", HEAD_GRAD, BT, Vp, d, bnc=False)}


@pytest.fixture(scope="module", autouse=True)
def built():
    from paper_2608_13578_amd import bcmt as abi
    if not os.path.exists(abi.LIB_PATH):
        from paper_2608_13578_amd.build import build
        build()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D", [64, 192, 2048])
@pytest.mark.parametrize("rows", [65535 * 64, 65535 * 64 + 1, 65535 * 128])
def test_grid_limits(dtype, D, rows):
    from paper_2608_13578_amd import bcmt as abi
    cfg = abi.make_config(1, rows, D, D // 64, rows, 0.8, dtype)
    assert abi.bcmt_validate(cfg) == abi.BCMT_OK
    for name, (kernel, (x, y, z), _) in layer_plans(1, rows, D, dtype).items():
        assert 1 <= x < 2 ** 31 and 1 <= y <= 65535 and 1 <= z <= 65535, (name, kernel, (x, y, z))


def test_every_kernel_is_reached():
    """The shapes the kernels were made for."""
    assert layer_plans(1, 256, 128, "f32")["qkv"][0] == F32_32
    assert layer_plans(4, 1024, 512, "f32")["qkv"][0] == F32_64
    assert layer_plans(1, 700, 768, "bf16")["score"][0] == PIPE_32
    p = layer_plans(8, 1024, 768, "bf16")
    assert (p["qkv"][0], p["score"][0], p["dx"][0]) == (PIPE_8, PIPE_8, PIPE_4)
    assert all(v[0] == WIDE for k, v in layer_plans(2, 65536, 1024, "bf16").items()
               if k in ("qkv", "score", "gate", "hbar", "dgrad", "dx"))


@pytest.mark.parametrize("M,D,residual,name,pipe_us,wide_us", [
    (12288, 1024, False, "gate", 41.7, 53.3),
    (24576, 1152, False, "gate", 89.2, 106.6),
    (65536, 384, True, "dx", 85.6, 102.5),
    (24576, 896, True, "dx", 137.3, 157.3),
    (20000, 1152, True, "dgrad", 59.4, 66.1),
    (24576, 1536, True, "score", 130.4, 139.0),
    (32768, 1024, True, "dx", 224.7, 171.4),
    (131072, 1024, True, "gate", 494.2, 456.3),
    (16384, 1024, True, "qkv", 107.7, 92.2),
])
def test_measured_products_run_on_the_faster_kernel(M, D, residual, name, pipe_us, wide_us):
    """Products of layers timed on 128 x 128 and on 256 x 256 tiles."""
    kernel = layer_plans(1, M, D, "bf16", residual)[name][0]
    assert (kernel == WIDE) == (wide_us < pipe_us)


@pytest.mark.parametrize("V,d,BT,name,pipe_us,wide_us", [
    (8000, 640, 16484, "gelu", 103.2, 144.0),
    (8000, 640, 16484, "gelu_bwd", 108.6, 147.7),
    (50257, 512, 16384, "gelu", 79.4, 95.4),
    (8000, 640, 16484, "stats", 203.2, 221.7),
    (8000, 640, 16484, "grad", 209.7, 247.0),
    (50257, 768, 4100, "stats", 416.6, 390.7),
    (50257, 768, 4100, "grad", 476.4, 430.4),
])
def test_measured_model_products_run_on_the_faster_kernel(V, d, BT, name, pipe_us, wide_us):
    kernel = model_plans(V, d, 1, BT)[name][0]
    assert (kernel == WIDE) == (wide_us < pipe_us)
