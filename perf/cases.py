"""Workloads of the BCMT library: what its users run, and in 64 bits what comes out.

Five kinds of call cover the public entry points:

  train    bcmt_layer_forward + bcmt_layer_backward (LayerBuffers), all
           parameter gradients: one layer of a training step;
  infer    bcmt_layer_forward without saved activations: a prompt or a batch
           that no backward follows;
  prefill  bcmt_layer_forward_chunk over consecutive chunks with the memory
           state handed on, no saved activations: a long prompt streamed in;
  chunks   chunked training: forward_chunk over the chunks, backward_chunk
           from the last to the first with accumulated weight gradients;
  decode   bcmt_decode_reset + one bcmt_decode_step per token of a block;
  lm       bcmt_model_train_step with AdamW: the language model's step.

Inputs are drawn on the GPU from the seed: activations and upstream gradients
N(0, 1), weights N(0, (0.55 / sqrt(D))^2) (the 0.02 of D = 768 at every
width), token ids with the skew of text.  They are rounded to the compute
type first, so that the 64-bit result starts from the same values.
"""

import math

import torch

from paper_2608_13578_amd import bcmt as abi
from paper_2608_13578_amd.layer import TORCH_DTYPE, DecodeBuffers, LayerBuffers, SideStream
from paper_2608_13578_amd.model import ModelBuffers

MATRICES = ("Wq", "Wk", "Wv", "Wo", "Wm", "Wg")
OPT = {"lr": 1e-4, "beta1": 0.9, "beta2": 0.999, "eps": 1e-8, "weight_decay": 0.01}


def _layer(name, kind, B, T, D, H, L, dtype="bf16", gamma=0.8, residual=False, channel=False,
           chunks=1):
    return {"name": name, "kind": kind, "B": B, "T": T, "D": D, "H": H, "L": L, "dtype": dtype,
            "gamma": gamma, "residual": residual, "channel": channel, "chunks": chunks}


def listed():
    return [
        # One sequence batch decoded in step through one block and its end:
        # serving, where each token is a handful of small launches.
        _layer("decode", "decode", 8, 128, 768, 12, 128, residual=True),
        # The smallest layer that is run in earnest: float32, a few blocks
        # (the package's own smoke test); launches and latency.
        _layer("small_f32", "train", 1, 256, 128, 2, 64, dtype="f32"),
        # One prompt of an odd length through one layer, no backward.
        _layer("infer_prompt", "infer", 1, 700, 768, 12, 128, residual=True),
        # A ragged batch: the last block is shorter than the others.
        _layer("train_ragged", "train", 2, 1000, 256, 4, 128, residual=True),
        # The paper's model width (8 heads of 16) at its small block size.
        _layer("train_paper", "train", 16, 1024, 128, 8, 64),
        # The measured layer: GPT-2-small width at the paper's context.
        _layer("train_layer", "train", 8, 1024, 768, 12, 128),
        # The dense limit of the block-size sweep: one block per sequence.
        _layer("train_dense", "train", 8, 1024, 768, 12, 1024),
        # Float32 training at an ordinary size.
        _layer("train_f32", "train", 4, 1024, 512, 8, 128, dtype="f32"),
        # Long-context training: 256 blocks per sequence.
        _layer("train_long", "train", 2, 65536, 1024, 16, 256, residual=True),
        # A long prompt streamed in as chunks of whole blocks.
        _layer("prefill_chunks", "prefill", 1, 16384, 1024, 16, 256, residual=True, chunks=4),
        # Chunked training with one decay per channel and many short blocks.
        _layer("train_chunks_channel", "chunks", 2, 16384, 768, 12, 64, channel=True, chunks=2),
        # The language model of the paper's experiments, one optimizer step.
        {"name": "lm_step", "kind": "lm", "V": 50257, "D": 128, "H": 8, "layers": 6, "B": 16,
         "T": 1024, "L": 128, "gamma": 0.8, "dtype": "bf16"},
    ]


def _log(rng, lo, hi):
    """A whole number in [lo, hi], spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _width(rng, lo, hi, heads):
    """(D, H): a model width (a multiple of 64, of 128 above 512, of 256
    above 1024) with heads of one of the given widths."""
    D = _log(rng, lo, hi)
    step = 64 if D <= 512 else 128 if D <= 1024 else 256
    D = max(lo, min(hi, (D + step // 2) // step * step))
    return D, D // rng.choice(heads)


def draw(rng):
    kind = rng.choice(["train", "train", "train", "infer", "prefill", "chunks", "decode", "lm"])
    gamma = round(rng.uniform(0.5, 0.95), 3)
    residual = rng.random() < 0.5
    channel = rng.random() < 0.25
    dtype = "f32" if rng.random() < 0.25 else "bf16"
    if kind == "lm":
        D = rng.choice([64, 128, 192, 256])
        T = _log(rng, 64, 1024)
        B = max(1, min(16, _log(rng, 512, 8192) // T))
        return {"kind": "lm", "V": _log(rng, 1000, 50257), "D": D, "H": D // rng.choice([16, 32]),
                "layers": rng.choice([1, 2, 4, 6]), "B": B, "T": T,
                "L": rng.choice([32, 64, 100, 128, 256, T]), "gamma": gamma, "dtype": "bf16"}
    if kind == "decode":
        D, H = _width(rng, 128, 1024, [64])
        L = _log(rng, 16, 128)
        c = _layer("", kind, _log(rng, 1, 64), L, D, H, L, dtype, gamma, residual, channel)
    else:
        D, H = _width(rng, 64, 1536, [64, 64, 32, 16])
        f32 = dtype == "f32"
        most = min(1 << 15 if f32 else 1 << 17, int((2e11 if f32 else 3e12) / (30.0 * D * D)))
        tokens = _log(rng, 64, most)
        B = _log(rng, 1, min(16, max(1, tokens // 32)))
        chunks = rng.choice([2, 3, 4]) if kind in ("prefill", "chunks") else 1
        T = max(1, tokens // B)
        L = _log(rng, 16, 1024 if not f32 else 256)
        if chunks > 1:  # chunks hold whole blocks; the sequence's last block may be short
            L = min(L, max(8, T // (2 * chunks)))
            T = max(T, chunks * L)
        c = _layer("", kind, B, T, D, H, L, dtype, gamma, residual, channel, chunks)
    del c["name"]
    return c


# ---------------------------------------------------------------- inputs

def _weights(c, gen):
    D = c["D"]
    dt = TORCH_DTYPE[c["dtype"]]

    def normal(*shape):
        w = torch.randn(*shape, generator=gen, device="cuda") * (0.55 / math.sqrt(D))
        return w.to(dt)
    W = {k: normal(D, D) for k in MATRICES}
    W["wp"] = normal(D)
    return W


def _decay(c, gen):
    """The decay: a number, or one per channel around it."""
    if not c["channel"]:
        return c["gamma"]
    g = torch.rand(c["D"], generator=gen, device="cuda") * 0.2 + (c["gamma"] - 0.1)
    return g.clamp(0.05, 0.97).cpu().numpy()


def _cuts(c):
    """Token ranges of the chunks: whole blocks each, the rest in the last."""
    T, L, n = c["T"], c["L"], c["chunks"]
    size = max(1, (-(-T // L)) // n) * L
    edges = [min(T, k * size) for k in range(n)] + [T]
    return [(a, b) for a, b in zip(edges, edges[1:]) if b > a]


def _inputs(c, seed):
    """(generator, weights, decay, X, dY): dY for the kinds with a backward;
    for decode X is [T, B, D], one step's input after another."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    W, decay = _weights(c, gen), _decay(c, gen)
    dt = TORCH_DTYPE[c["dtype"]]
    shape = (c["T"], c["B"], c["D"]) if c["kind"] == "decode" else (c["B"], c["T"], c["D"])
    X = torch.randn(shape, generator=gen, device="cuda").to(dt)
    dY = torch.randn(shape, generator=gen, device="cuda").to(dt) if c["kind"] in ("train", "chunks") else None
    return gen, W, decay, X, dY


def _state(c, gen, decay):
    """A memory state (N, Z) as many blocks of history leave it."""
    B, D = c["B"], c["D"]
    g = torch.as_tensor(decay, dtype=torch.float32, device="cuda")
    Z = (1 / (1 - g)).expand(B, D).contiguous() if c["channel"] else (1 / (1 - g)).repeat(B)
    m = torch.randn(B, D, generator=gen, device="cuda") * 0.1
    return m * (Z if c["channel"] else Z[:, None]), Z


def _grads(c):
    """Gradient buffers; the short ones (dwp and the decay's) back to back."""
    D = c["D"]
    g = {"d" + k: torch.zeros(D, D, device="cuda") for k in MATRICES}
    g["short"] = torch.zeros(D + (D if c["channel"] else 4), device="cuda")
    args = {k: v for k, v in g.items() if k != "short"}
    args["dwp"] = g["short"][:D]
    args["dgamma_ch" if c["channel"] else "dgamma"] = g["short"][D:]
    if c["channel"]:
        args["dgamma"] = None
    return g, args


def _buffers(c, W, decay, T, accumulate=False, side=True):
    lb = LayerBuffers(c["B"], T, c["D"], c["H"], c["L"], gamma=decay, dtype=c["dtype"],
                      residual=c["residual"], accumulate=accumulate, side=side)
    lb.params = dict(W)
    if lb.gamma_ch is not None:
        lb.params["gamma_ch"] = lb.gamma_ch
    return lb


def _lm_inputs(c, seed):
    """(flat float32 parameters as a function of the layout, tokens, targets)."""
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def params(names, layout, n):
        p = torch.randn(n, generator=gen, device="cuda") * 0.02
        for name, (off, cnt) in zip(names, layout):
            if name.endswith("_g"):
                p[off:off + cnt] = 1.0
            elif name.endswith("_b"):
                p[off:off + cnt] = 0.0
            elif name == "E":
                p[off + c["V"] * c["D"]:off + cnt] = 0.0
        return p
    # ranks as in text: the r-th most frequent token about as often as 1 / r
    u = torch.rand(c["B"], c["T"] + 1, generator=gen, device="cuda", dtype=torch.float64)
    ids = ((c["V"] + 1.0) ** u - 1.0).long().clamp(0, c["V"] - 1).int()
    return params, ids[:, :-1].contiguous(), ids[:, 1:].contiguous()


def prepare(case, seed):
    c = case
    if c["kind"] == "lm":
        params, tokens, targets = _lm_inputs(c, seed)
        mb = ModelBuffers(c["V"], c["D"], c["H"], c["layers"], c["B"], c["T"], c["L"], c["gamma"])
        mb.params.copy_(params(mb.names, mb.layout, mb.n))
        abi.bcmt_model_cast(mb.cfg, mb.params, mb.params_bf16)
        return {"case": c, "mb": mb, "tokens": tokens, "targets": targets}
    gen, W, decay, X, dY = _inputs(c, seed)
    s = {"case": c, "X": X, "dY": dY}
    if c["kind"] == "decode":
        db = DecodeBuffers(c["B"], c["D"], c["H"], c["L"], gamma=decay, dtype=c["dtype"],
                           residual=c["residual"])
        db.params = dict(W)
        if db.gamma_ch is not None:
            db.params["gamma_ch"] = db.gamma_ch
        s.update(db=db, carry=_state(c, gen, decay), y=torch.empty_like(X))
        return s
    if c["kind"] == "train":
        lb = _buffers(c, W, decay, c["T"])
        s["grads"], s["args"] = _grads(c)
        s.update(lb=lb, Y=lb.new_activation(), dX=lb.new_activation())
        return s
    if c["kind"] == "infer":
        lb = _buffers(c, W, decay, c["T"], side=None)
        s.update(cfg=lb.cfg, params=lb.params, Y=lb.new_activation(),
                 ws=_workspace(lb.cfg))
        return s
    cuts = _cuts(c)
    side = SideStream() if c["kind"] == "chunks" else None
    runs = []
    for k, (a, b) in enumerate(cuts):
        lb = _buffers(c, W, decay, b - a, accumulate=k + 1 < len(cuts), side=side)
        r = {"lb": lb, "X": X[:, a:b].contiguous(), "Y": lb.new_activation(),
             "carry": lb.new_carry()}
        if c["kind"] == "chunks":
            r.update(dY=dY[:, a:b].contiguous(), dX=lb.new_activation(), dcarry=lb.new_carry())
        else:
            lb.saved = None
            r["ws"] = _workspace(lb.cfg)
        runs.append(r)
    s = {"case": c, "runs": runs}
    if c["kind"] == "chunks":
        s["grads"], s["args"] = _grads(c)
    return s


def _workspace(cfg):
    n = abi.bcmt_workspace_bytes(cfg, abi.BCMT_PASS_INFERENCE)
    return torch.empty(max(256, n), dtype=torch.uint8, device="cuda")


def run(state):
    s = state
    kind = s["case"]["kind"]
    if kind == "train":
        s["lb"].forward(s["X"], s["Y"])
        s["lb"].backward(s["X"], s["dY"], s["dX"], s["args"])
        return {"Y": s["Y"], "dX": s["dX"], **s["grads"]}
    if kind == "infer":
        abi.bcmt_layer_forward(s["cfg"], s["X"], s["params"], s["Y"], None, s["ws"])
        return {"Y": s["Y"]}
    if kind == "decode":
        db, X, y = s["db"], s["X"], s["y"]
        db.reset(s["carry"])
        for t in range(s["case"]["T"]):
            db.step(t, X[t], y[t])
        return {"y": y}
    if kind == "lm":
        mb = s["mb"]
        mb.step(s["tokens"], s["targets"], OPT)
        return {"loss": mb.loss, "grads": mb.grads, "params": mb.params, "m": mb.m, "v": mb.v}
    carry = None
    for r in s["runs"]:
        if kind == "prefill":
            lb = r["lb"]
            abi.bcmt_layer_forward_chunk(lb.cfg, r["X"], lb.params, carry, r["Y"], r["carry"],
                                         None, r["ws"])
        else:
            r["lb"].forward_chunk(r["X"], r["Y"], carry, r["carry"])
        carry = r["carry"]
    out = {"Y": [r["Y"] for r in s["runs"]], "N": carry[0], "Z": carry[1]}
    if kind == "chunks":
        dcarry = None
        for r in reversed(s["runs"]):
            r["lb"].backward_chunk(r["X"], r["dY"], dcarry, r["dX"], r["dcarry"], s["args"])
            dcarry = r["dcarry"]
        out.update(dX=[r["dX"] for r in s["runs"]], **s["grads"])
    return out


# ---------------------------------------------------------------- what it cannot do without

def _pairs(T, L):
    """Causal query-key pairs of one sequence's blocks."""
    full, rest = divmod(T, L)
    return full * (L * (L + 1) // 2) + rest * (rest + 1) // 2


def _forward_flops(B, T, D, L):
    nb = -(-T // L)
    return 10 * B * T * D * D + 2 * B * nb * D * D + 4 * B * D * _pairs(T, L)


def work(case):
    c = case
    B, T, D, L = c["B"], c["T"], c["D"], c["L"]
    if c["kind"] == "lm":
        n = c["V"] * D + T * D + c["layers"] * (14 * D * D + 5 * D) + 2 * D
        fwd = c["layers"] * (_forward_flops(B, T, D, L) + 16 * B * T * D * D) + 2 * B * T * D * c["V"]
        # float32 weights and moments read and written, gradients written
        return {"flops": 3 * fwd, "bytes": 28 * n + 8 * B * T}
    es = 4 if c["dtype"] == "f32" else 2
    weights, act = 6 * D * D, B * T * D
    if c["kind"] == "decode":  # every step reads the weights; the state stays small
        flops = T * B * 10 * D * D + 4 * B * D * _pairs(T, T) + 4 * B * D * D
        return {"flops": flops, "bytes": (T * 5 * D * D + D * D) * es + 2 * act * es}
    fwd = _forward_flops(B, T, D, L)
    if c["kind"] in ("infer", "prefill"):
        return {"flops": fwd, "bytes": (weights * len(_cuts(c)) + 2 * act) * es}
    return {"flops": 3 * fwd, "bytes": (weights + 4 * act) * es + weights * 4}


def tolerance(case):
    """About four times the start's distance from the 64-bit result, over
    150 drawn cases (largest seen: forward outputs 3.6e-3, one element
    4.5e-2; gradients 6.6e-3 and 1.5e-2 for those of wp and the decay, small
    sums of large terms, one element 0.14; the language model 7.8e-3 and
    0.32; float32 2.3e-6 and 1.1e-5)."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    if case["kind"] in ("infer", "prefill", "decode"):
        return {"rel": 0.015, "max": 0.2}
    return {"rel": 0.03, "max": 0.9 if case["kind"] == "lm" else 0.5}


# ---------------------------------------------------------------- in 64 bits

def _layer64(X, W, gamma, L, H, residual, state=None):
    """The layer in float64: (Y, N, Z) for X [B, T, D]; gamma a tensor, one
    value or one per channel; state the incoming (N [B, D], Z [B, 1] or
    [B, D]), None for none."""
    B, T, D = X.shape
    dh, nb = D // H, -(-T // L)
    Lb = min(L, T)
    pad = nb * Lb - T

    def heads(x):
        x = torch.nn.functional.pad(x, (0, 0, 0, pad))
        return x.reshape(B, nb, Lb, H, dh).transpose(2, 3).reshape(-1, Lb, dh).contiguous()
    causal = torch.ones(Lb, Lb, dtype=torch.bool, device=X.device).tril()
    s = torch.bmm(heads(X @ W["Wq"]), heads(X @ W["Wk"]).transpose(1, 2).contiguous())
    s = (s / math.sqrt(dh)).masked_fill(~causal, -math.inf)
    o = torch.bmm(torch.softmax(s, -1), heads(X @ W["Wv"]))
    o = o.reshape(B, nb, H, Lb, dh).transpose(2, 3).reshape(B, nb * Lb, D)[:, :T]
    Hl = o @ W["Wo"]
    Hb = torch.nn.functional.pad(Hl, (0, 0, 0, pad)).reshape(B, nb, Lb, D)
    there = (torch.arange(nb * Lb, device=X.device) < T).reshape(nb, Lb)
    a = torch.softmax((Hb @ W["wp"]).masked_fill(~there, -math.inf), -1)
    S = (a[..., None] * Hb).sum(2)
    if state is None:
        N, Z = torch.zeros_like(S[:, 0]), torch.zeros_like(S[:, 0])
        ms = [torch.zeros_like(N)]
    else:
        N, Z = state[0], state[1].expand(B, D)
        ms = [N / Z]
    for i in range(nb):
        N, Z = gamma * N + S[:, i], gamma * Z + 1
        ms.append(N / Z)
    C = torch.stack(ms[:-1], 1) @ W["Wm"]
    C = C[:, :, None].expand(B, nb, Lb, D).reshape(B, nb * Lb, D)[:, :T]
    Y = Hl + torch.sigmoid(Hl @ W["Wg"]) * C
    return (X + Y if residual else Y), N, Z


def _exact_lm(c, seed):
    params, tokens, targets = _lm_inputs(c, seed)
    cfg = abi.make_model_config(c["V"], c["D"], c["H"], c["layers"], c["B"], c["T"], c["L"],
                                c["gamma"])
    d, nl = c["D"], c["layers"]
    from paper_2608_13578_amd.inputs import model_array_names
    names = model_array_names(nl)
    layout = [abi.bcmt_model_param_array(cfg, i) for i in range(len(names))]
    p32 = params(names, layout, abi.bcmt_model_param_count(cfg))
    flat = torch.empty(p32.numel(), dtype=torch.float64, device="cuda")
    for name, (off, cnt) in zip(names, layout):
        v = p32[off:off + cnt]
        ln = name.endswith("_g") or name.endswith("_b")
        flat[off:off + cnt] = (v if ln else v.bfloat16()).double()
    flat.requires_grad_(True)
    P = {n: flat[off:off + cnt] for n, (off, cnt) in zip(names, layout)}
    gamma = torch.tensor(c["gamma"], dtype=torch.float32).double().cuda()

    def norm(x, k):
        return torch.nn.functional.layer_norm(x, (d,), P[k + "_g"], P[k + "_b"], 1e-5)
    E = P["E"].reshape(-1, d)
    x = E[tokens.long()] + P["Pe"].reshape(-1, d)[None]
    for i in range(nl):
        W = {k: P["%d.%s" % (i, k)].reshape(d, d) for k in MATRICES}
        W["wp"] = P["%d.wp" % i]
        x = x + _layer64(norm(x, "%d.ln1" % i), W, gamma, c["L"], c["H"], False)[0]
        u = norm(x, "%d.ln2" % i) @ P["%d.W1" % i].reshape(d, 4 * d)
        x = x + torch.nn.functional.gelu(u, approximate="tanh") @ P["%d.W2" % i].reshape(4 * d, d)
    z = norm(x, "lnf").reshape(-1, d) @ E[:c["V"]].t()
    loss = torch.nn.functional.cross_entropy(z, targets.long().reshape(-1))
    loss.backward()
    g = flat.grad
    m, v = (1 - OPT["beta1"]) * g, (1 - OPT["beta2"]) * g * g
    p = p32.double() * (1 - OPT["lr"] * OPT["weight_decay"])
    p = p - OPT["lr"] * g / (g.abs() + OPT["eps"])
    return {"loss": loss.detach().reshape(1), "grads": g, "params": p, "m": m, "v": v}


def exact(case, seed):
    c = case
    if c["kind"] == "lm":
        return _exact_lm(c, seed)
    gen, W, decay, X, dY = _inputs(c, seed)
    W = {k: v.double().requires_grad_(dY is not None) for k, v in W.items()}
    gamma = torch.as_tensor(decay, dtype=torch.float32).double().cuda().requires_grad_(dY is not None)
    if c["kind"] == "decode":
        N, Z = (t.double() for t in _state(c, gen, decay))
        Y, _, _ = _layer64(X.double().transpose(0, 1).contiguous(), W, gamma, c["L"], c["H"],
                           c["residual"], (N, Z if c["channel"] else Z[:, None]))
        return {"y": Y.transpose(0, 1).contiguous()}
    X = X.double().requires_grad_(dY is not None)
    Y, N, Z = _layer64(X, W, gamma, c["L"], c["H"], c["residual"])
    cuts = _cuts(c)
    out = {"Y": Y.detach()}
    if c["kind"] in ("prefill", "chunks"):
        out = {"Y": [Y[:, a:b].detach().contiguous() for a, b in cuts], "N": N.detach(),
               "Z": Z.detach().contiguous() if c["channel"] else Z[:, 0].detach().contiguous()}
    if dY is not None:
        Y.backward(dY.double())
        dX = X.grad
        out["dX"] = [dX[:, a:b].contiguous() for a, b in cuts] if c["kind"] == "chunks" else dX
        # a single block uses neither Wm nor Wg nor the decay: zero gradients
        g = {k: torch.zeros_like(v) if v.grad is None else v.grad
             for k, v in {**W, "gamma": gamma}.items()}
        out.update({"d" + k: g[k] for k in MATRICES})
        dg = g["gamma"].reshape(-1)
        if not c["channel"]:
            dg = torch.nn.functional.pad(dg, (0, 3))
        out["short"] = torch.cat([g["wp"], dg])
    return out
