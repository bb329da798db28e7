"""What a training step of a model under stochastic backpropagation asks of this library, as cases to be timed.

A case is a dict of plain values.  Six kinds of work, each as a user's program runs it through the Python entry points:

  linear      one Linear / pointwise-conv layer: draw the keep-set, cache the kept rows of the input, backward
  step        the independent linears of a block in the batched calls (one draw, one cache call, one backward call)
  block       a transformer block as the dependent chain it is in a model: cache the kept rows of what the backward
              needs, then fc2, GELU, fc1, LayerNorm, proj, attention, qkv, LayerNorm backward on compact rows
  conv_block  a ConvNeXt block as a chain: layer scale, pw2, GELU, pw1, LayerNorm, depthwise 7 x 7 backward
  downsample  a p x p, stride p down-sampling layer: cache patch rows, linear backward, scatter
  attention   the attention core's backward on the kept tokens alone

Values: activations, gradients N(0, 1), weights N(0, 0.02^2), scales around 1, as in synth_inputs.py; the attention
output and the row log-sum-exp come from an ordinary softmax over all tokens of the sample.
"""
import math

import torch

import paper_2210_00129_amd as sbp

DT = {"bf16": torch.bfloat16, "f32": torch.float32}
MODES = {"grid": sbp.GRID_PER_CELL, "random": sbp.RANDOM_MASK}
VIT_BASE = "768x2304,768x768,768x3072,3072x768"


def listed():
    return [
        # One layer of a unit-test-sized fp32 model (64 -> 256 on two 14 x 14 maps): launches and host time are everything.
        dict(name="linear_small_f32", kind="linear", dtype="f32", B=2, P=0, H=14, W=14, k=2, Cin=64, Cout=256, dw_bf16=False,
             accumulate=False),
        # A classifier-like layer on an odd map with channel counts that fill no tile, weight gradient kept in bf16.
        dict(name="linear_ragged", kind="linear", dtype="bf16", B=9, P=1, H=13, W=17, k=3, Cin=200, Cout=1000, dw_bf16=True,
             accumulate=False),
        # One wide layer of a large model (16384 kept rows of 32768, 4096 x 4096): the largest call.
        dict(name="linear_wide", kind="linear", dtype="bf16", B=128, P=0, H=16, W=16, k=2, Cin=4096, Cout=4096, dw_bf16=False,
             accumulate=False),
        # The MLP of ViT-Tiny in the batched calls: small layers, latency-bound.
        dict(name="step_vit_tiny", kind="step", dtype="bf16", B=64, P=1, H=14, W=14, k=2, mode="grid", layers="192x768,768x192",
             accumulate=False),
        # The four linears of a ViT-Base block in the batched calls: the headline workload of the benchmark.
        dict(name="step_vit_base", kind="step", dtype="bf16", B=64, P=1, H=14, W=14, k=2, mode="grid", layers=VIT_BASE,
             accumulate=False),
        # The pointwise convs of a ConvNeXt-B detection stage 2 with the random-mask sampler, gradients accumulated over
        # micro-batches.
        dict(name="step_det_s2_random", kind="step", dtype="bf16", B=2, P=0, H=100, W=168, k=2, mode="random",
             layers="256x1024,1024x256", accumulate=True),
        # A whole ViT-Base block, every layer waiting for the one before it: what a model's backward really runs.
        dict(name="block_vit_base", kind="block", dtype="bf16", B=64, P=1, H=14, W=14, k=2, heads=12, d=64),
        # A ViT-Tiny block (3 heads of 64) trained in fp32.
        dict(name="block_vit_tiny_f32", kind="block", dtype="f32", B=64, P=1, H=14, W=14, k=2, heads=3, d=64),
        # The ConvNeXt-B stage-3 block of a detector (50 x 84 x 512): short launches in a chain.
        dict(name="conv_block_s3", kind="conv_block", dtype="bf16", B=2, H=50, W=84, k=2, C=512),
        # The stage-1 block (200 x 336 x 128) at keep ratio 1/4: streaming.
        dict(name="conv_block_s1", kind="conv_block", dtype="bf16", B=2, H=200, W=336, k=1, C=128),
        # The down-sampling layer between stages 1 and 2 (2 x 2, stride 2, 128 -> 256 channels).
        dict(name="downsample_s1", kind="downsample", dtype="bf16", B=2, H=200, W=336, p=2, k=2, C=128, Cout=256),
        # The attention core with many tokens per sample (1024 kept of 2048).
        dict(name="attention_long", kind="attention", dtype="bf16", B=8, n=2048, n_k=1024, heads=12, d=64),
    ]


# ---- drawn cases --------------------------------------------------------------------------------------------------
def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    """A channel count: mostly a multiple of 64 or 8 as models have them, now and then any number."""
    c = _log(rng, lo, hi)
    step = rng.choice((64, 64, 64, 8, 8, 1))
    return max(step, c // step * step)


def _draw_linear(rng):
    f32 = rng.random() < 0.3
    c = dict(kind="linear", dtype="f32" if f32 else "bf16", B=_log(rng, 1, 128), P=rng.choice((0, 1)), H=rng.randint(7, 32),
             W=rng.randint(7, 32), k=rng.randint(1, 4), Cin=_channels(rng, 64, 768 if f32 else 4096),
             Cout=_channels(rng, 64, 768 if f32 else 4096), dw_bf16=rng.random() < 0.25, accumulate=False)
    c["accumulate"] = not c["dw_bf16"] and rng.random() < 0.25
    return c


def _draw_step(rng):
    if rng.random() < 0.5:
        C = 64 * rng.randint(3, 16)
        side = rng.choice((7, 14, 14, 16, rng.randint(7, 20)))
        c = dict(B=_log(rng, 4, 128), P=1, H=side, W=side, layers=f"{C}x{3 * C},{C}x{C},{C}x{4 * C},{4 * C}x{C}")
    else:
        C = 32 * rng.randint(3, 20)
        c = dict(B=rng.randint(1, 4), P=0, H=_log(rng, 14, 200), W=_log(rng, 14, 336), layers=f"{C}x{4 * C},{4 * C}x{C}")
    return dict(kind="step", dtype="bf16", **c, k=rng.randint(1, 4), mode=rng.choice(("grid", "grid", "grid", "random")),
                accumulate=rng.random() < 0.25)


def _draw_block(rng):
    f32 = rng.random() < 0.3
    side = rng.randint(7, 16)
    return dict(kind="block", dtype="f32" if f32 else "bf16", B=_log(rng, 2, 64), P=rng.choice((0, 1)), H=side, W=side,
                k=rng.randint(1, 4), heads=rng.randint(2, 4) if f32 else rng.randint(3, 16), d=rng.choice((32, 64, 64)))


def _draw_conv_block(rng):
    return dict(kind="conv_block", dtype="bf16", B=rng.randint(1, 4), H=_log(rng, 13, 200), W=_log(rng, 13, 336),
                k=rng.randint(1, 4), C=32 * rng.randint(3, 24))


def _draw_downsample(rng):
    p = rng.choice((2, 2, 2, 4))
    C = 32 * rng.randint(2, 12)
    return dict(kind="downsample", dtype="bf16", B=rng.randint(1, 4), H=p * _log(rng, 10, 100), W=p * _log(rng, 10, 168), p=p,
                k=rng.randint(1, 4), C=C, Cout=2 * C)


def _draw_attention(rng):
    n_k = _log(rng, 32, 1536)
    return dict(kind="attention", dtype="bf16", B=_log(rng, 1, 64), n=n_k * rng.choice((1, 2, 4)), n_k=n_k,
                heads=rng.randint(2, 16), d=rng.choice((32, 64, 64, 128)))


DRAWS = (_draw_linear, _draw_linear, _draw_step, _draw_step, _draw_block, _draw_block, _draw_conv_block, _draw_conv_block,
         _draw_downsample, _draw_attention)
# The largest listed work of a kind and type: no drawn case asks for more of either.
_CAPS = {}


def draw(rng):
    if not _CAPS:
        for c in listed():
            key, w = (c["kind"], c["dtype"]), work(c)
            old = _CAPS.get(key, (0, 0))
            _CAPS[key] = (max(old[0], w["bytes"]), max(old[1], w["flops"]))
        _CAPS[("linear", "f32")] = _CAPS[("block", "f32")]
    make = rng.choice(DRAWS)
    while True:
        c = make(rng)
        w, cap = work(c), _CAPS[(c["kind"], c["dtype"])]
        if w["bytes"] <= cap[0] and w["flops"] <= cap[1] and max(c.get("n", 0), 1) <= 4096:
            return c


# ---- sizes and work ---------------------------------------------------------------------------------------------------
def _layers(c):
    return [tuple(int(v) for v in s.split("x")) for s in c["layers"].split(",")]


def _rows(c):
    """(rows M, kept rows K) of the case's map."""
    P, H, W = c.get("P", 0), c["H"], c["W"]
    if c["kind"] == "downsample":
        H, W = H // c["p"], W // c["p"]
    mode = MODES[c.get("mode", "grid")]
    return c["B"] * (P + H * W), sbp.keep_count(c["B"], P, H, W, c["k"], mode)


def _linear_work(K, Cin, Cout, s, dw):
    """(bytes, flops) of one linear backward on compact rows: dY_k, X_k, W in; dW, db, dX_k out."""
    return s * (K * Cout + K * Cin + Cin * Cout) + dw * Cin * Cout + 4 * Cout + s * K * Cin, 4 * K * Cin * Cout


def work(case):
    c = case
    s = 2 if c["dtype"] == "bf16" else 4
    if c["kind"] == "attention":
        rows, hd = c["B"] * c["n_k"], c["heads"] * c["d"]
        return {"bytes": 8 * s * rows * hd + 4 * rows * c["heads"], "flops": 10 * c["B"] * c["heads"] * c["n_k"] ** 2 * c["d"]}
    M, K = _rows(c)
    nbytes, flops = 4 * (K + M), 0                        # idx and inv
    if c["kind"] in ("linear", "step"):
        for Cin, Cout in [(c["Cin"], c["Cout"])] if c["kind"] == "linear" else _layers(c):
            dw = (2 if c.get("dw_bf16") else 4) * (2 if c["accumulate"] else 1)
            b, f = _linear_work(K, Cin, Cout, s, dw)
            nbytes += b + s * (M - K) * Cin + s * K * Cin  # the dropped rows of dX; X_k is written
            flops += f
    elif c["kind"] == "block":
        C = c["heads"] * c["d"]
        # kept rows read once: x1, u1, qkv, a, x2, u2, z, the output gradient, lse; written: dX
        nbytes += s * K * (3 * C + C + C + C + C + C + 4 * C + C) + 4 * K * c["heads"] + s * M * C
        nbytes += (s + 4) * 12 * C * C + 4 * 9 * C + 4 * 6 * C   # weights in, their gradients out; db; LayerNorm scales
        n_k = K // c["B"]
        flops += 4 * K * 12 * C * C + 10 * c["B"] * c["heads"] * n_k * n_k * c["d"]
    elif c["kind"] == "conv_block":
        C = c["C"]
        nbytes += s * K * (C + C + C + 4 * C + C) + 2 * s * M * C + (s + 4) * (8 * C * C + 49 * C) + 4 * 12 * C
        flops += 4 * K * 8 * C * C + 4 * 49 * K * C
    else:                                                  # downsample
        Cin = c["p"] ** 2 * c["C"]
        b, f = _linear_work(K, Cin, c["Cout"], s, 4)
        nbytes += b + s * (M - K) * Cin + s * K * Cin      # dX at full size; the patch rows are written
        flops += f
    return {"bytes": nbytes, "flops": flops}


# ---- inputs ------------------------------------------------------------------------------------------------------------
class _Values:
    def __init__(self, dtype, seed):
        self.dtype, self.g = dtype, torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def __call__(self, *shape, std=1.0):
        return torch.randn(*shape, generator=self.g, device="cuda").mul_(std).to(self.dtype)

    def weight(self, *shape):
        return self(*shape, std=0.02)

    def scale(self, C):
        return 1.0 + 0.1 * torch.randn(C, generator=self.g, device="cuda")


def _attention_forward(qkv, B, n, h, d):
    """(attention output [B n, h d], row log-sum-exp [B n, h]) of the model's forward over all n tokens."""
    A = torch.empty(B * n, h * d, dtype=qkv.dtype, device="cuda")
    lse = torch.empty(B * n, h, device="cuda")
    for b in range(B):
        q, k, v = qkv[b * n:(b + 1) * n].float().view(n, 3, h, d).permute(1, 2, 0, 3).contiguous()
        m = torch.matmul(q, k.transpose(1, 2).contiguous()) * d ** -0.5
        lse[b * n:(b + 1) * n] = torch.logsumexp(m, -1).t()
        A[b * n:(b + 1) * n] = torch.matmul(torch.softmax(m, -1), v).permute(1, 0, 2).reshape(n, h * d).to(qkv.dtype)
    return A, lse


def prepare(case, seed):
    c = case
    v = _Values(DT[c["dtype"]], seed)
    st = {"case": c, "seed": seed}
    if c["kind"] == "attention":
        B, n, n_k, h, d = c["B"], c["n"], c["n_k"], c["heads"], c["d"]
        qkv = v(B * n, 3 * h * d)
        A, lse = _attention_forward(qkv, B, n, h, d)
        keep = torch.stack([torch.randperm(n, generator=v.g, device="cuda")[:n_k].sort()[0] + b * n for b in range(B)]).view(-1)
        st.update(qkv=qkv[keep], A=A[keep], lse=lse[keep], dA=v(B * n_k, h * d))
        return st
    M, K = _rows(c)
    st.update(M=M, K=K)
    if c["kind"] == "linear":
        st.update(X=v(M, c["Cin"]), W=v.weight(c["Cout"], c["Cin"]), dY=v(M, c["Cout"]), flags=0)
        if c["dw_bf16"]:
            st["flags"] |= sbp.FLAG_DW_OUT_BF16
        if c["accumulate"]:                                # gradients of the micro-batches before
            st["flags"] |= sbp.FLAG_ACCUMULATE_DW
            st.update(dW=torch.zeros(c["Cout"], c["Cin"], device="cuda"), db=torch.zeros(c["Cout"], device="cuda"))
    elif c["kind"] == "step":
        # the program keeps its output buffers and one workspace
        flags = sbp.FLAG_ACCUMULATE_DW if c["accumulate"] else 0
        idx = torch.empty(K, dtype=torch.int32, device="cuda")
        inv = torch.empty(M, dtype=torch.int32, device="cuda")
        Xs, Xks, layers = [], [], []
        for Cin, Cout in _layers(c):
            Xs.append(v(M, Cin))
            Xks.append(torch.empty(K, Cin, dtype=v.dtype, device="cuda"))
            layers.append(dict(dY=v(M, Cout), idx=idx, inv=inv, X_k=Xks[-1], W=v.weight(Cout, Cin), M=M, flags=flags,
                               dW=torch.zeros(Cout, Cin, device="cuda"), db=torch.zeros(Cout, device="cuda"),
                               dX=torch.empty(M, Cin, dtype=v.dtype, device="cuda")))
        descs = [sbp.make_layer(**l) for l in layers]
        need = sbp.backward_linear_batch_workspace(descs, sbp.BF16 if c["dtype"] == "bf16" else sbp.F32)
        st.update(idx=idx, inv=inv, Xs=Xs, Xks=Xks, layers=layers,
                  ws=torch.empty(max(need, 256), dtype=torch.uint8, device="cuda"))
    elif c["kind"] == "block":
        C, h, d, B = c["heads"] * c["d"], c["heads"], c["d"], c["B"]
        qkv = v(M, 3 * C)
        A, lse = _attention_forward(qkv, B, M // B, h, d)
        st.update(qkv=qkv, A=A, lse=lse, x1=v(M, C), u1=v(M, C), x2=v(M, C), u2=v(M, C), z=v(M, 4 * C), dOut=v(M, C),
                  Wqkv=v.weight(3 * C, C), Wproj=v.weight(C, C), W1=v.weight(4 * C, C), W2=v.weight(C, 4 * C),
                  g1=v.scale(C), g2=v.scale(C))
    elif c["kind"] == "conv_block":
        C = c["C"]
        st.update(X=v(c["B"], c["H"], c["W"], C), y=v(M, C), u=v(M, C), z=v(M, 4 * C), s=v(M, C), dOut=v(M, C),
                  Wd=v.weight(7, 7, C), W1=v.weight(4 * C, C), W2=v.weight(C, 4 * C), g=v.scale(C), gls=v.scale(C))
    else:
        st.update(X=v(c["B"], c["H"], c["W"], c["C"]), dY=v(M, c["Cout"]), W=v.weight(c["Cout"], c["p"] ** 2 * c["C"]))
    return st


# ---- the passes ----------------------------------------------------------------------------------------------------------
COMPACT = sbp.FLAG_DY_COMPACT | sbp.FLAG_DX_COMPACT


def _run_linear(st):
    c = st["case"]
    idx, inv = sbp.sample_indices(c["B"], c["P"], c["H"], c["W"], c["k"], st["seed"], 1, want_inv=True)
    Xk = sbp.forward_cache(st["X"], idx)
    dW, db, dX = sbp.backward_linear(st["dY"], idx, Xk, st["W"], inv=inv, flags=st["flags"], dW=st.get("dW"), db=st.get("db"))
    return {"idx": idx, "inv": inv, "Xk": Xk, "dW": dW, "db": db, "dX": dX}


def _run_step(st):
    c = st["case"]
    sbp.sample_indices(c["B"], c["P"], c["H"], c["W"], c["k"], st["seed"], 1, mode=MODES[c["mode"]], idx_out=st["idx"],
                       inv_out=st["inv"])
    sbp.forward_cache_batch(st["Xs"], [st["idx"]] * len(st["Xs"]), outs=st["Xks"])
    out = sbp.backward_linear_batch(st["layers"], workspace=st["ws"])
    return {"idx": st["idx"], "inv": st["inv"], "Xks": st["Xks"], "grads": out}


def _run_block(st):
    c, M = st["case"], st["M"]
    idx, inv = sbp.sample_indices(c["B"], c["P"], c["H"], c["W"], c["k"], st["seed"], 1, want_inv=True)
    names = ("x1", "u1", "qkv", "A", "x2", "u2", "z")
    x1, u1, qkv, A, x2, u2, z = sbp.forward_cache_batch([st[n] for n in names], [idx] * len(names))
    lse = sbp.forward_cache(st["lse"], idx)
    dO = sbp.forward_cache(st["dOut"], idx)
    H = sbp.act_forward_rows(z)
    dW2, db2, dH = sbp.backward_linear(dO, idx, H, st["W2"], M=M, flags=COMPACT)
    dZ = sbp.act_backward_rows(dH, z, out=dH)
    dW1, db1, dU2 = sbp.backward_linear(dZ, idx, u2, st["W1"], M=M, flags=COMPACT)
    dg2, dbeta2, dx2 = sbp.backward_layernorm(dU2, x2, st["g2"], 1e-6, idx, M, flags=sbp.FLAG_DX_COMPACT)
    dR = dO + dx2                                          # the residual around the MLP
    dWp, dbp, dA = sbp.backward_linear(dR, idx, A, st["Wproj"], M=M, flags=COMPACT)
    dqkv = sbp.backward_attention(qkv, A, dA, lse, c["B"], c["heads"], c["d"], c["d"] ** -0.5)
    dWq, dbq, dU1 = sbp.backward_linear(dqkv, idx, u1, st["Wqkv"], M=M, flags=COMPACT)
    dg1, dbeta1, dX = sbp.backward_layernorm(dU1, x1, st["g1"], 1e-6, idx, M, inv=inv)
    return {"idx": idx, "inv": inv, "dW": [dW2, dW1, dWp, dWq], "db": [db2, db1, dbp, dbq], "dg": [dg2, dg1],
            "dbeta": [dbeta2, dbeta1], "dX": dX}


def _run_conv_block(st):
    c, M = st["case"], st["M"]
    B, H, W, C = st["X"].shape
    idx, inv = sbp.sample_indices(B, 0, H, W, c["k"], st["seed"], 1, want_inv=True)
    y, u, z, s, dO = sbp.forward_cache_batch([st["y"], st["u"], st["z"], st["s"], st["dOut"]], [idx] * 5)
    dgls, dS = sbp.backward_layerscale(dO, s, st["gls"])
    Hk = sbp.act_forward_rows(z)
    dW2, db2, dH = sbp.backward_linear(dS, idx, Hk, st["W2"], M=M, flags=COMPACT)
    dZ = sbp.act_backward_rows(dH, z, out=dH)
    dW1, db1, dU = sbp.backward_linear(dZ, idx, u, st["W1"], M=M, flags=COMPACT)
    dg, dbeta, dY = sbp.backward_layernorm(dU, y, st["g"], 1e-6, idx, M, inv=inv)
    dWd, dbd, dX = sbp.backward_dwconv(dY.view(B, H, W, C), idx, st["X"], st["Wd"], inv=inv)
    return {"idx": idx, "inv": inv, "dW": [dW2, dW1, dWd], "db": [db2, db1, dbd], "dg": [dgls, dg], "dbeta": dbeta, "dX": dX}


def _run_downsample(st):
    c, p = st["case"], st["case"]["p"]
    B, H, W, C = st["X"].shape
    idx, inv = sbp.sample_indices(B, 0, H // p, W // p, c["k"], st["seed"], 1, want_inv=True)
    Xk = sbp.forward_cache_patches(st["X"], idx, p)
    dW, db, dXp = sbp.backward_linear(st["dY"], idx, Xk, st["W"], flags=sbp.FLAG_DX_COMPACT, inv=inv)
    dX = sbp.scatter_patches(dXp, idx, (B, H, W, C), p, inv=inv)
    return {"idx": idx, "inv": inv, "Xk": Xk, "dW": dW, "db": db, "dX": dX}


def _run_attention(st):
    c = st["case"]
    return {"dqkv": sbp.backward_attention(st["qkv"], st["A"], st["dA"], st["lse"], c["B"], c["heads"], c["d"], c["d"] ** -0.5)}


RUNS = {"linear": _run_linear, "step": _run_step, "block": _run_block, "conv_block": _run_conv_block,
        "downsample": _run_downsample, "attention": _run_attention}


def run(state):
    return RUNS[state["case"]["kind"]](state)


def tolerance(case):
    """Keep-sets and gathered rows are the same bits.  Largest errors of the gradients against the same passes in 64 bits
    (2-norm; largest element over the root mean square or the value): fp32 chains 6e-7, 5e-6; single steps with outputs
    rounded to bf16 once 1.7e-3, 3.9e-3 (that rounding); bf16 chains and attention, which round between their steps,
    4.3e-3, 3.4e-2.  About four times these (fp32: more, for sums over many more rows)."""
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 1e-4}
    if case["kind"] in ("block", "conv_block", "attention"):
        return {"rel": 1.7e-2, "max": 1.4e-1}
    return {"rel": 6.6e-3, "max": 1.6e-2}
