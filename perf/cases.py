"""The work that a user of this library has it do, as timed cases.

Five kinds of work, each through the public binding (paper_2309_14717_amd.api):

  step      one adapted linear in fine-tuning: forward and backward (dx, dA, dB)
  mlp       a LLaMA MLP block in fine-tuning: gate and up as one wide layer that shares x, SwiGLU,
            down; forward and backward
  forward   the merged (adapter-free) layer in serving, from one token to a long prompt
  quantize  codes and factors of a weight: min-max, or error-compensated under a Hessian
  adamw     the optimiser step over the adapters of one decoder layer

Shapes are those of the benchmark configurations (LLaMA layer shapes) and sizes between them.
Weights ~ N(0, 0.02), activations ~ N(0, 1) with a few outlier channels, everything made on the
device from the seed.
"""
import math

import torch

from paper_2309_14717_amd import api

DEV = "cuda"


def listed():
    return [
        # A small adapted layer on a short sequence: the smallest training call, launches and latency count.
        dict(name="step_small", kind="step", tokens=64, d_in=1024, d_out=1024, bits=4, group=32, rank=16, s=2.0,
             keep=True, bf16=False, accumulate=False),
        # A 7B attention projection at a 4096-token batch: the benchmark's default workload.
        dict(name="step_attention", kind="step", tokens=4096, d_in=4096, d_out=4096, bits=4, group=32, rank=64, s=0.25,
             keep=True, bf16=True, accumulate=False),
        # A 13B MLP projection with 3-bit codes on an odd token count, gradients accumulated over
        # micro-batches, the backward reading x again instead of kept pooled activations.
        dict(name="step_int3_ragged", kind="step", tokens=1531, d_in=5120, d_out=13824, bits=3, group=64, rank=64, s=0.25,
             keep=False, bf16=True, accumulate=True),
        # The 7B MLP block at a 4096-token batch.
        dict(name="mlp_block", kind="mlp", tokens=4096, d_in=4096, d_mid=11008, bits=4, group=32, rank=64, s=0.25),
        # Decoding one sequence on a merged 65B model: both MLP shapes from the deployment stream.
        dict(name="decode_1", kind="forward", tokens=1, d_in=8192, d_out=22016, bits=4, group=32, pair=True,
             layout="deployed", bf16=True),
        # Decoding sixteen sequences at once on the quantized triple.
        dict(name="decode_16", kind="forward", tokens=16, d_in=8192, d_out=22016, bits=4, group=32, pair=True,
             layout="triple", bf16=True),
        # Decoding a batch of sixty-four sequences (or a short prompt): between the streaming
        # kernels and full tiles.
        dict(name="batch_64", kind="forward", tokens=64, d_in=8192, d_out=22016, bits=4, group=32, pair=True,
             layout="triple", bf16=True),
        # A 256-token prompt on the deployed layer.
        dict(name="prompt_256", kind="forward", tokens=256, d_in=8192, d_out=22016, bits=4, group=32, pair=True,
             layout="deployed", bf16=True),
        # A prompt of odd length on a 13B layer with 2-bit codes, fp32 result.
        dict(name="prompt_int2", kind="forward", tokens=700, d_in=5120, d_out=13824, bits=2, group=64, pair=False,
             layout="triple", bf16=False),
        # Quantizing a 7B MLP weight by min-max.
        dict(name="quantize", kind="quantize", d_in=4096, d_out=11008, bits=4, group=32, compensated=False),
        # Quantizing a 7B attention weight with error compensation.
        dict(name="quantize_compensated", kind="quantize", d_in=4096, d_out=4096, bits=4, group=32, compensated=True),
        # The optimiser step over the 14 adapter tensors of a 7B decoder layer.
        dict(name="adamw", kind="adamw", d_in=4096, d_mid=11008, group=32, rank=64),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mult(rng, lo, hi, unit):
    return max(lo, _log(rng, lo, hi) // unit * unit)


def draw(rng):
    kind = rng.choice(["step", "step", "step", "forward", "forward", "forward", "forward", "mlp", "quantize", "quantize",
                       "adamw"])
    bits = rng.choice([4, 4, 4, 3, 2])
    group = rng.choice([32, 32, 64, 128])
    rank = rng.choice([8, 16, 32, 64, 64, 128])
    if kind == "step":
        # layers of 512 .. 13824 features; widths that are multiples of eight only among them
        while True:
            tokens = _log(rng, 16, 4096)
            d_in = _mult(rng, 512, 13824, 128)
            d_out = _mult(rng, 512, 13824, rng.choice([8, 64, 128]))
            if tokens * d_in * d_out <= 4096 * 4096 * 11008:
                break
        return dict(kind=kind, tokens=tokens, d_in=d_in, d_out=d_out, bits=bits, group=group, rank=rank, s=0.25,
                    keep=rng.random() < 0.6, bf16=rng.random() < 0.7, accumulate=rng.random() < 0.4)
    if kind == "mlp":
        return dict(kind=kind, tokens=_log(rng, 64, 4096), d_in=_mult(rng, 1024, 4096, 128),
                    d_mid=_mult(rng, 2048, 11008, 128), bits=bits, group=group, rank=rank, s=0.25)
    if kind == "forward":
        layout = rng.choice(["triple", "triple", "deployed", "factors16"])
        if layout == "deployed":
            bits = 4
        pair = rng.random() < 0.5
        d_out = _mult(rng, 1024, 22016, 128 if pair else rng.choice([8, 64, 128]))
        return dict(kind=kind, tokens=_log(rng, 1, 1024), d_in=_mult(rng, 1024, 8192, 128), d_out=d_out, bits=bits,
                    group=group, pair=pair, layout=layout, bf16=rng.random() < 0.7)
    if kind == "quantize":
        if rng.random() < 0.5:
            return dict(kind=kind, d_in=_mult(rng, 512, 4096, group), d_out=_mult(rng, 512, 4096, 8), bits=bits, group=group,
                        compensated=True)
        return dict(kind=kind, d_in=_mult(rng, 1024, 8192, group), d_out=_mult(rng, 1024, 22016, 8), bits=bits, group=group,
                    compensated=False)
    return dict(kind=kind, d_in=_mult(rng, 1024, 8192, 128), d_mid=_mult(rng, 2048, 22016, 128), group=group, rank=rank)


# ---- inputs -------------------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _normal(gen, shape, std=1.0, dtype=torch.float32):
    return (torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32) * std).to(dtype)


def _activations(gen, tokens, width):
    x = _normal(gen, (tokens, width))
    n = width // 1000  # a few channels are much larger than the rest, as in LLaMA activations
    if n:
        x[:, torch.randint(0, width, (n,), generator=gen, device=DEV)] *= 20.0
    return x.to(torch.bfloat16)


def _weight(gen, d_in, d_out):
    return _normal(gen, (d_in, d_out), 0.02)


def _adapter(gen, d_in, d_out, group, rank):
    return _normal(gen, (d_in // group, rank), 0.02), _normal(gen, (rank, d_out), 0.02)


def _hessian_factor(gen, n):
    """The upper Cholesky factor of the inverse Hessian of correlated calibration inputs."""
    x = _normal(gen, (2 * n, n), dtype=torch.float64)
    x[:, 1:] += 0.5 * x[:, :-1].clone()
    h = x.T @ x / (2 * n)
    h.diagonal().add_(0.01 * h.diagonal().mean())
    inv = torch.cholesky_inverse(torch.linalg.cholesky(h))
    return torch.linalg.cholesky(inv, upper=True).float().contiguous()


def _layers(case):
    """The linears of a "forward" case, as (d_in, d_out)."""
    shape = (case["d_in"], case["d_out"])
    return [shape, shape[::-1]] if case["pair"] else [shape]


def _forward_inputs(case, gen):
    for d_in, d_out in _layers(case):
        W = _weight(gen, d_in, d_out)
        A, B = _adapter(gen, d_in, d_out, case["group"], 64)
        yield d_in, d_out, W, (0.25 / case["group"]) * (A @ B), _activations(gen, case["tokens"], d_in)


def _step_inputs(case, gen):
    d_in, d_out, T = case["d_in"], case["d_out"], case["tokens"]
    W = _weight(gen, d_in, d_out)
    A, B = _adapter(gen, d_in, d_out, case["group"], case["rank"])
    x = _activations(gen, T, d_in)
    dy = _normal(gen, (T, d_out), dtype=torch.bfloat16)
    return W, A, B, x, dy, _normal(gen, tuple(A.shape)), _normal(gen, tuple(B.shape))


def _mlp_inputs(case, gen):
    d, m, g, r, T = case["d_in"], case["d_mid"], case["group"], case["rank"], case["tokens"]
    W_gu, W_d = _weight(gen, d, 2 * m), _weight(gen, m, d)
    ads = [_adapter(gen, d, m, g, r), _adapter(gen, d, m, g, r), _adapter(gen, m, d, g, r)]
    return W_gu, W_d, ads, _activations(gen, T, d), _normal(gen, (T, d), dtype=torch.bfloat16)


def _adamw_shapes(case):
    d, m, g, r = case["d_in"], case["d_mid"], case["group"], case["rank"]
    return [s for i, o in [(d, d)] * 4 + [(d, m)] * 2 + [(m, d)] for s in ((i // g, r), (r, o))]


def _adamw_inputs(case, gen):
    shapes = _adamw_shapes(case)
    return ([_normal(gen, s, 0.02) for s in shapes], [_normal(gen, s, 0.01) for s in shapes],
            [_normal(gen, s, 0.001) for s in shapes], [_normal(gen, s, 0.01).square() for s in shapes])


_HP = dict(lr=2e-5, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01, max_grad_norm=0.3)
_STEP = 11


def _ws(nbytes):
    return torch.empty(max(int(nbytes), 4096), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    gen, kind = _gen(seed), case["kind"]
    st = {"case": case}
    if kind == "step":
        W, A, B, x, dy, dA, dB = _step_inputs(case, gen)
        desc = api.make_desc(case["d_in"], case["d_out"], case["bits"], case["group"], case["rank"], case["s"])
        T = case["tokens"]
        st.update(desc=desc, triple=api.quantize(desc, W), A=A, B=B, x=x, dy=dy,
                  dtype=torch.bfloat16 if case["bf16"] else torch.float32,
                  ws=_ws(max(api.workspace_bytes(desc, T, api.OP_FORWARD), api.workspace_bytes(desc, T, api.OP_BACKWARD))))
        # an accumulating backward adds to what the gradients hold: this micro-batch starts from them
        st.update(dA0=dA, dB0=dB, dA=dA.clone(), dB=dB.clone())
    elif kind == "mlp":
        W_gu, W_d, ads, x, dy = _mlp_inputs(case, gen)
        d, m, T = case["d_in"], case["d_mid"], case["tokens"]
        gu = api.make_desc(d, 2 * m, case["bits"], case["group"], 0, 0.0)
        down = api.make_desc(m, d, case["bits"], case["group"], case["rank"], case["s"])
        adapters = [(A, B, case["s"]) for A, B in ads[:2]]
        grads = [(torch.zeros_like(A), torch.zeros_like(B)) for A, B in ads]
        parts = api._parts(gu, adapters, x.device)
        size = lambda op: int(api.load().qalora_shared_workspace_bytes(gu, T, op, 2, parts))  # noqa: E731
        st.update(gu=gu, down=down, t_gu=api.quantize(gu, W_gu), t_d=api.quantize(down, W_d), adapters=adapters,
                  down_ad=ads[2], x=x, dy=dy, grads=grads,
                  ws=_ws(max(size(api.OP_FORWARD), size(api.OP_BACKWARD), api.workspace_bytes(down, T, api.OP_FORWARD),
                             api.workspace_bytes(down, T, api.OP_BACKWARD))))
    elif kind == "forward":
        st["dtype"] = torch.bfloat16 if case["bf16"] else torch.float32
        layers, size = [], 0
        op = api.OP_FORWARD_FACTORS16 if case["layout"] == "factors16" else api.OP_FORWARD
        for d_in, d_out, W, shift, x in _forward_inputs(case, gen):
            desc = api.make_desc(d_in, d_out, case["bits"], case["group"])
            packed, alpha, beta = api.quantize(desc, W)
            beta = beta + shift
            held = None
            if case["layout"] == "deployed":
                held = api.deploy(desc, packed, alpha, beta)
            elif case["layout"] == "factors16":
                held = api.pack_factors16(desc, alpha, beta)
            layers.append((desc, x, packed, alpha, beta, held))
            size = max(size, api.workspace_bytes(desc, case["tokens"], op))
        st.update(layers=layers, ws=_ws(size))
    elif kind == "quantize":
        desc = api.make_desc(case["d_in"], case["d_out"], case["bits"], case["group"])
        st.update(desc=desc, W=_weight(gen, case["d_in"], case["d_out"]))
        if case["compensated"]:
            st["U"] = _hessian_factor(gen, case["d_in"])
    else:
        p, g, m, v = _adamw_inputs(case, gen)
        numel = [t.numel() for t in p]
        size = api.load().qalora_adamw_workspace_bytes(len(p), (api.ctypes.c_size_t * len(p))(*numel))
        st.update(hp=api.AdamW(**_HP), p=p, g=g, m=m, v=v,
                  norm=torch.zeros(1, dtype=torch.float32, device=DEV), ws=_ws(size), step=_STEP)
    return st


# ---- one pass -----------------------------------------------------------------------------------

def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "step":
        d, t, ws, dt = st["desc"], st["triple"], st["ws"], st["dtype"]
        acc = case["accumulate"]
        dA, dB = st["dA"], st["dB"]
        if acc:  # the previous micro-batch's gradients, so that every pass starts from the same ones
            dA.copy_(st["dA0"])
            dB.copy_(st["dB0"])
        if case["keep"]:
            y, kept = api.forward_keep(d, st["x"], *t, st["A"], st["B"], out_dtype=dt, ws=ws)
            dx, dA, dB = api.backward_kept(d, st["dy"], kept, *t, st["A"], st["B"], dx_dtype=dt, dA=dA, dB=dB,
                                           accumulate=acc, ws=ws)
        else:
            y = api.forward(d, st["x"], *t, st["A"], st["B"], out_dtype=dt, ws=ws)
            dx, dA, dB = api.backward(d, st["dy"], st["x"], *t, st["A"], st["B"], dx_dtype=dt, dA=dA, dB=dB,
                                      accumulate=acc, ws=ws)
        return [y, dx, dA, dB]
    if kind == "mlp":
        m, ws, bf = case["d_mid"], st["ws"], torch.bfloat16
        gu, kept = api.forward_shared(st["gu"], st["x"], *st["t_gu"], st["adapters"], keep=True, out_dtype=bf, ws=ws)
        h = api.swiglu_forward_strided(gu, m)
        A, B = st["down_ad"]
        y, kept_d = api.forward_keep(st["down"], h, *st["t_d"], A, B, out_dtype=bf, ws=ws)
        dA, dB = st["grads"][2]
        dh, dA, dB = api.backward_kept(st["down"], st["dy"], kept_d, *st["t_d"], A, B, dx_dtype=bf, dA=dA, dB=dB, ws=ws)
        dgu = api.swiglu_backward_strided(dh, gu, m)
        dx, grads = api.backward_shared(st["gu"], dgu, None, kept, *st["t_gu"], st["adapters"], dx_dtype=bf,
                                        grads=st["grads"][:2], ws=ws)
        return [y, dx, dA, dB] + [t for pair in grads for t in pair]
    if kind == "forward":
        out = []
        for desc, x, packed, alpha, beta, held in st["layers"]:
            if case["layout"] == "deployed":
                out.append(api.forward_deployed(desc, x, held, packed, out_dtype=st["dtype"], ws=st["ws"]))
            elif case["layout"] == "factors16":
                out.append(api.forward_factors16(desc, x, packed, held, out_dtype=st["dtype"], ws=st["ws"]))
            else:
                out.append(api.forward(desc, x, packed, alpha, beta, out_dtype=st["dtype"], ws=st["ws"]))
        return out
    if kind == "quantize":
        if case["compensated"]:
            return list(api.quantize_compensated(st["desc"], st["W"], st["U"]))
        return list(api.quantize(st["desc"], st["W"]))
    api.adamw_step(st["hp"], st["step"], st["p"], st["g"], st["m"], st["v"], grad_norm=st["norm"], ws=st["ws"])
    return {"p": st["p"], "m": st["m"], "v": st["v"], "norm": st["norm"]}


# ---- what a pass cannot do without --------------------------------------------------------------

def _layer_bytes(d_in, d_out, bits, group):
    """Codes and the two fp32 factors of a layer."""
    return d_in * d_out * bits / 8 + 8 * (d_in // group) * d_out


def work(case):
    kind = case["kind"]
    if kind == "step":
        T, i, o, g, r = case["tokens"], case["d_in"], case["d_out"], case["group"], case["rank"]
        es, ad = (2 if case["bf16"] else 4), (i // g * r + r * o) * 4
        layer = _layer_bytes(i, o, case["bits"], g)
        # forward and backward each read the layer and the adapter; x and dy are read, y and dx written
        nbytes = 2 * (layer + ad) + T * (i + o) * 2 + T * (i + o) * es + ad * (2 if case["accumulate"] else 1)
        # two dense contractions; adapter: P A, U B, dy B^T, U^T dy, P^T dU, dU A^T
        flops = 4 * T * i * o + 6 * T * r * (i // g + o)
        return {"bytes": nbytes, "flops": flops}
    if kind == "mlp":
        T, d, m, g, r, b = (case[k] for k in ("tokens", "d_in", "d_mid", "group", "rank", "bits"))
        ad = 4 * (2 * (d // g * r + r * m) + m // g * r + r * d)
        nbytes = 2 * (_layer_bytes(d, 2 * m, b, g) + _layer_bytes(m, d, b, g)) + 3 * ad + 2 * T * 4 * d
        flops = 12 * T * d * m + 6 * T * r * (2 * (d // g + m) + m // g + d)
        return {"bytes": nbytes, "flops": flops}
    if kind == "forward":
        T, es = case["tokens"], 2 if case["bf16"] else 4
        nbytes = flops = 0
        for i, o in _layers(case):
            fac = (i // case["group"]) * o * (4 if case["layout"] == "factors16" else 8)
            nbytes += i * o * case["bits"] / 8 + fac + T * i * 2 + T * o * es
            flops += 2 * T * i * o
        return {"bytes": nbytes, "flops": flops}
    if kind == "quantize":
        i, o = case["d_in"], case["d_out"]
        nbytes = 4 * i * o + _layer_bytes(i, o, case["bits"], case["group"])
        if case["compensated"]:
            # every row's error goes to all later rows: half of d_in x d_in multiply-adds per column
            return {"bytes": nbytes + 2 * i * i, "flops": i * i * o}
        return {"bytes": nbytes, "flops": 5 * i * o}
    n = sum(a * b for a, b in _adamw_shapes(case))
    return {"bytes": 28 * n, "flops": 14 * n}


def tolerance(case):
    if case["kind"] == "quantize":
        return "exact"  # the recipe fixes the order of its fp32 operations: codes and factors bit for bit
    if case["kind"] == "adamw":
        return {"rel": 1e-6}
    if case["kind"] == "mlp":
        return {"rel": 1.4e-2}
    if case["bf16"]:
        return {"rel": 7e-3}
    if case["kind"] == "forward" and case["tokens"] <= (32 if case["bits"] == 4 else 16):
        return {"rel": 5e-6}
    return {"rel": 2e-3}


# ---- the same in 64 bits ------------------------------------------------------------------------

def _quantized(W, bits, group):
    """Eq. 1 per group of rows and column, in the fp32 recipe: codes, alpha, beta."""
    d_in, d_out = W.shape
    w = W.view(d_in // group, group, d_out)
    beta = w.amin(1)
    alpha = (w.amax(1) - beta) / float(2 ** bits - 1)
    alpha = torch.where(alpha > 0, alpha, torch.full_like(alpha, 2.0 ** -60))
    codes = ((w - beta[:, None]) / alpha[:, None]).round().clamp(0, 2 ** bits - 1)
    return codes.view(d_in, d_out), alpha, beta


def _weight64(W, bits, group, shift=None, fp16=False):
    codes, alpha, beta = _quantized(W, bits, group)
    if shift is not None:
        beta = beta + shift
    if fp16:
        alpha, beta = alpha.half(), beta.half()
    rows = lambda t: t.double().repeat_interleave(group, 0)  # noqa: E731
    return codes.double() * rows(alpha) + rows(beta)


def _pool64(x, group):
    return x.view(x.shape[0], -1, group).mean(2)


def _linear64(x, Wq, A, B, s, group):
    return x @ Wq + s * (_pool64(x, group) @ A) @ B


def _linear_backward64(dy, x, Wq, A, B, s, group):
    P = _pool64(x, group)
    dU = s * (dy @ B.T)
    dx = dy @ Wq.T + (dU @ A.T).repeat_interleave(group, 1) / group
    return dx, P.T @ dU, s * (P @ A).T @ dy


def exact(case, seed):
    gen, kind, D = _gen(seed), case["kind"], torch.float64
    if kind == "step":
        W, A, B, x, dy, dA0, dB0 = _step_inputs(case, gen)
        Wq = _weight64(W, case["bits"], case["group"])
        A, B, x, dy = A.to(D), B.to(D), x.to(D), dy.to(D)
        y = _linear64(x, Wq, A, B, case["s"], case["group"])
        dx, dA, dB = _linear_backward64(dy, x, Wq, A, B, case["s"], case["group"])
        if case["accumulate"]:
            dA, dB = dA + dA0, dB + dB0
        return [y, dx, dA, dB]
    if kind == "mlp":
        W_gu, W_d, ads, x, dy = _mlp_inputs(case, gen)
        m, g, s, b = case["d_mid"], case["group"], case["s"], case["bits"]
        ads, x, dy = [(A.to(D), B.to(D)) for A, B in ads], x.to(D), dy.to(D)
        Wg, Wu, Wd = _weight64(W_gu[:, :m], b, g), _weight64(W_gu[:, m:], b, g), _weight64(W_d, b, g)
        gate, up = (_linear64(x, Wq, A, B, s, g) for Wq, (A, B) in ((Wg, ads[0]), (Wu, ads[1])))
        sig = torch.sigmoid(gate)
        h = gate * sig * up
        y = _linear64(h, Wd, *ads[2], s, g)
        dh, dA, dB = _linear_backward64(dy, h, Wd, *ads[2], s, g)
        dgate, dup = dh * up * sig * (1 + gate * (1 - sig)), dh * gate * sig
        dxg, dAg, dBg = _linear_backward64(dgate, x, Wg, *ads[0], s, g)
        dxu, dAu, dBu = _linear_backward64(dup, x, Wu, *ads[1], s, g)
        return [y, dxg + dxu, dA, dB, dAg, dBg, dAu, dBu]
    if kind == "forward":
        out = []
        for d_in, d_out, W, shift, x in _forward_inputs(case, gen):
            out.append(x.to(D) @ _weight64(W, case["bits"], case["group"], shift, case["layout"] == "factors16"))
        return out
    if kind == "quantize":
        if case["compensated"]:
            return None  # d_in dependent rows; and a code that rounds otherwise in 64 bits changes all rows behind it
        W = _weight(gen, case["d_in"], case["d_out"]).to(D)
        w = W.view(-1, case["group"], case["d_out"])
        lo, hi = w.amin(1), w.amax(1)
        return [None, (hi - lo) / (2 ** case["bits"] - 1), lo]
    # the first pass on a new state (the state is updated in place); hyperparameters as the fp32 they are given as
    hp = {k: float(torch.tensor(v, dtype=torch.float32)) for k, v in _HP.items()}
    p, g, m, v = ([t.to(D) for t in ts] for ts in _adamw_inputs(case, gen))
    norm = torch.sqrt(sum(t.square().sum() for t in g))
    clip = torch.clamp(hp["max_grad_norm"] / (norm + 1e-6), max=1.0)
    g = [t * clip for t in g]
    m = [hp["beta1"] * a + (1 - hp["beta1"]) * b for a, b in zip(m, g)]
    v = [hp["beta2"] * a + (1 - hp["beta2"]) * b * b for a, b in zip(v, g)]
    c1, c2 = 1 - hp["beta1"] ** _STEP, 1 - hp["beta2"] ** _STEP
    p = [a * (1 - hp["lr"] * hp["weight_decay"]) - hp["lr"] * (b / c1) / (torch.sqrt(c / c2) + hp["eps"])
         for a, b, c in zip(p, m, v)]
    return {"p": p, "m": m, "v": v, "norm": norm.view(1)}
