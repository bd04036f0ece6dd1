"""GPU parity on the degenerate and extreme cases of the layer: one token, one group per column,
the largest supported rank, token rows of wildly different magnitude (each row has its own
power-of-two scale inside the kernels, so a row-wise comparison is the meaningful one), the
split-K configuration of the dense kernel, and adapters that are exactly zero."""
import numpy as np
import pytest
import torch

import oracle
from paper_2309_14717_amd import synth
from helpers import TOL, dev, layer_on_gpu, record, rel_err

pytestmark = pytest.mark.gpu


def cfg_of(**kw):
    base = dict(name="edge", tokens=64, d_in=512, d_out=264, bits=4, group=32, rank=16, s=0.5, seed=21)
    base.update(kw)
    return synth.LayerConfig(**base)


def run_both(gpu_api, cfg, inputs=None):
    L = layer_on_gpu(gpu_api, cfg, inputs=inputs)
    d = L["np"]
    y = gpu_api.forward(L["desc"], L["x"], L["packed"], L["g_alpha"], L["g_beta"], L["A"], L["B"])
    dx, dA, dB = gpu_api.backward(L["desc"], L["dy"], L["x"], L["packed"], L["g_alpha"], L["g_beta"],
                                  L["A"], L["B"])
    ry = oracle.forward(d["x"], L["codes"], L["alpha"], L["beta"], cfg.group, d["A"], d["B"], cfg.s)
    rdx, rdA, rdB = oracle.backward(d["dy"], d["x"], L["codes"], L["alpha"], L["beta"], cfg.group,
                                    d["A"], d["B"], cfg.s)
    got = dict(y=y, dx=dx, dA=dA, dB=dB)
    ref = dict(y=ry, dx=rdx, dA=rdA, dB=rdB)
    return L, {k: v.cpu().numpy() for k, v in got.items()}, ref


def test_single_token_with_adapter(gpu_api):
    """T = 1 with an adapter takes the dense kernel (one ragged row tile), forward and backward."""
    cfg = cfg_of(tokens=1)
    _, got, ref = run_both(gpu_api, cfg)
    errs = {k: rel_err(got[k], ref[k]) for k in got}
    record("edge T=1 adapter", **errs)
    assert max(errs.values()) <= TOL


@pytest.mark.parametrize("bits", [2, 3, 4])
def test_one_group_per_column(gpu_api, bits):
    """L = 1 (Sec. 3.3's column-wise case): group = d_in, the adapter's A is a single row."""
    cfg = cfg_of(bits=bits, d_in=256, group=256, tokens=40, rank=8)
    _, got, ref = run_both(gpu_api, cfg)
    errs = {k: rel_err(got[k], ref[k]) for k in got}
    record(f"edge L=1 bits={bits}", **errs)
    # a 256-row group at 2 bits has a coarse grid: operand rounding is still what bounds it
    assert max(errs.values()) <= TOL


def test_one_short_group_per_column(gpu_api):
    """K = 64 in a single group: the roundings of a column's one (alpha, beta) pair act on all of
    its terms alike.  The matrix path evaluates alpha * (c - mid) + (beta + mid * alpha), whose
    constant term is small, and stays well inside the bar (about 4e-4 here)."""
    cfg = cfg_of(bits=4, d_in=64, group=64, d_out=776, tokens=257, rank=64, s=1.0, seed=32136)
    L, got, ref = run_both(gpu_api, cfg)
    errs = {k: rel_err(got[k], ref[k]) for k in got}
    bm = gpu_api.merge(L["desc"], L["g_beta"], L["A"], L["B"])
    ym = gpu_api.forward(L["desc"], L["x"], L["packed"], L["g_alpha"], bm)
    errs["y_merged"] = rel_err(ym.cpu().numpy(), ref["y"])
    record("edge L=1 K=64", **errs)
    assert max(errs.values()) <= 0.5 * TOL


@pytest.mark.parametrize("bits", [2, 3, 4])
def test_constant_groups_through_matrix_path(gpu_api, bits):
    """Groups whose weights are all equal (codes 0, the placeholder step) among ordinary ones.
    One-hot token rows read W~ back row by row: a constant group must come back as its value to
    fp16 rounding (2^-11 relative), whatever form the kernel evaluates alpha * c + beta in."""
    cfg = cfg_of(bits=bits, d_in=256, group=32, d_out=72, tokens=256, rank=0)
    d = synth.make_inputs(cfg)
    vals = np.array([0.0237, -0.4161, 3.3e-3, 117.3, -0.0, 1.0], np.float32)
    for n, v in enumerate(vals):
        d["W"][32 * n:32 * (n + 1), 5 * n + 1] = v
    d["x"] = np.eye(256, dtype=np.float32)
    L = layer_on_gpu(gpu_api, cfg, inputs=d)
    assert all(L["alpha"][n, 5 * n + 1] == np.float32(2.0 ** -60) for n in range(len(vals)))
    y = gpu_api.forward(L["desc"], L["x"], L["packed"], L["g_alpha"], L["g_beta"]).cpu().numpy()
    dx = gpu_api.backward(L["desc"], L["x"][:, :72].contiguous(), L["x"], L["packed"], L["g_alpha"],
                          L["g_beta"])[0].cpu().numpy()
    Wt = oracle.dequantize(L["codes"], L["alpha"], L["beta"], cfg.group)
    assert rel_err(y, Wt) <= TOL
    for n, v in enumerate(vals):
        got = y[32 * n:32 * (n + 1), 5 * n + 1].astype(np.float64)
        assert np.abs(got - float(v)).max() <= 2.0 ** -11 * abs(float(v)), (n, v, got[:4])
        # dy = the first 72 one-hot rows: dx[j, :] = W~[:, j], the same weights through the backward
        got_b = dx[5 * n + 1, 32 * n:32 * (n + 1)].astype(np.float64)
        assert np.abs(got_b - float(v)).max() <= 2.0 ** -11 * abs(float(v)), (n, v, got_b[:4])


def test_largest_rank(gpu_api):
    cfg = cfg_of(rank=128, tokens=150, d_out=520)
    _, got, ref = run_both(gpu_api, cfg)
    errs = {k: rel_err(got[k], ref[k]) for k in got}
    record("edge rank=128", **errs)
    assert max(errs.values()) <= TOL


def test_rows_of_very_different_magnitude(gpu_api):
    """Token rows scaled by 2^-100 ... 2^+100 and one all-zero row.  Every row carries its own
    power-of-two scale through the kernels, so each row must meet the bar on its own."""
    cfg = cfg_of(tokens=48, rank=16)
    d = synth.make_inputs(cfg)
    rng = np.random.default_rng(5)
    exps = rng.integers(-100, 101, cfg.tokens)
    exps[:4] = [-100, 100, 0, 37]
    scale = np.ldexp(1.0, exps).astype(np.float32)[:, None]
    d["x"] = (d["x"] * scale).astype(np.float32)      # powers of two keep bf16 representability
    d["dy"] = (d["dy"] * scale[::-1]).astype(np.float32)
    d["x"][7] = 0.0
    d["dy"][9] = 0.0
    L, got, ref = run_both(gpu_api, cfg, inputs=d)
    for name in ("y", "dx"):
        g, r = got[name].astype(np.float64), ref[name]
        assert np.isfinite(g).all()
        row_max = np.abs(r).max(axis=1)
        err = np.abs(g - r).max(axis=1)
        ok = err <= TOL * row_max
        assert ok.all(), (name, np.nonzero(~ok)[0][:5], (err / np.maximum(row_max, 1e-300))[~ok][:5])
    assert (got["y"][7] == got["y"][7]).all()
    # x row 7 is zero: y row 7 is exactly zero; dy row 9 is zero: dx row 9 is exactly zero
    assert not got["y"][7].any() and not got["dx"][9].any()


def test_split_k_dense_path(gpu_api):
    """Few column tiles and a long K: the dense kernel splits K over block rows and a second
    launch adds the slices in order.  fp32 and bf16 outputs, with and without the adapter."""
    cfg = cfg_of(tokens=200, d_in=2048, d_out=256, rank=24)
    L, got, ref = run_both(gpu_api, cfg)
    errs = {k: rel_err(got[k], ref[k]) for k in got}
    record("edge split-K T=200 2048x256", **errs)
    assert max(errs.values()) <= TOL
    a = (L["desc"], L["x"], L["packed"], L["g_alpha"], L["g_beta"], L["A"], L["B"])
    y32 = gpu_api.forward(*a)
    y16 = gpu_api.forward(*a, out_dtype=torch.bfloat16)
    assert torch.equal(y16, y32.to(torch.bfloat16))
    assert torch.equal(y32, gpu_api.forward(*a))
    y0 = gpu_api.forward(L["desc"], L["x"], L["packed"], L["g_alpha"], L["g_beta"])
    r0 = oracle.forward(L["np"]["x"], L["codes"], L["alpha"], L["beta"], cfg.group)
    assert rel_err(y0.cpu().numpy(), r0) <= TOL


def test_zero_adapter_matches_adapter_free(gpu_api):
    """B = 0 (the usual initialisation): the adapted forward equals the adapter-free one bit
    for bit, dA is exactly zero and dB is not."""
    cfg = cfg_of(tokens=130)
    d = synth.make_inputs(cfg)
    d["B"] = np.zeros_like(d["B"])
    L = layer_on_gpu(gpu_api, cfg, inputs=d)
    y_ad = gpu_api.forward(L["desc"], L["x"], L["packed"], L["g_alpha"], L["g_beta"], L["A"], L["B"])
    y_free = gpu_api.forward(L["desc"], L["x"], L["packed"], L["g_alpha"], L["g_beta"])
    assert torch.equal(y_ad, y_free)
    _, dA, dB = gpu_api.backward(L["desc"], L["dy"], L["x"], L["packed"], L["g_alpha"], L["g_beta"],
                                 L["A"], L["B"])
    assert not dA.any().item()
    _, _, rdB = oracle.backward(d["dy"], d["x"], L["codes"], L["alpha"], L["beta"], cfg.group,
                                d["A"], d["B"], cfg.s, want_dx=False)
    assert rel_err(dB.cpu().numpy(), rdB) <= TOL and dB.abs().max().item() > 0


def test_binding_rejects_mismatched_tensors(gpu_api):
    """The C ABI sees raw pointers only, so the binding checks every operand's shape, dtype and
    device against the descriptor before marshalling: a mismatch is an exception, never an
    out-of-bounds access on the device."""
    cfg = synth.LayerConfig("val", 8, 256, 64, 4, 32, 8, 0.5, seed=3)
    L = layer_on_gpu(gpu_api, cfg)
    ok = (L["desc"], L["x"], L["packed"], L["g_alpha"], L["g_beta"], L["A"], L["B"])
    gpu_api.forward(*ok)
    bad_cases = [
        (L["desc"], L["x"][:, :128].contiguous(), *ok[2:]),          # x narrower than d_in
        (L["desc"], L["x"].float(), *ok[2:]),                        # x not bf16
        (L["desc"], L["x"], L["packed"][:-16], *ok[3:]),             # packed too short
        (L["desc"], L["x"], L["packed"], L["g_alpha"][:-1], *ok[4:]),  # alpha short of a group row
        (L["desc"], L["x"], L["packed"], L["g_alpha"], L["g_beta"].double(), L["A"], L["B"]),
        (*ok[:5], L["A"][:, :4].contiguous(), L["B"]),               # A of the wrong rank
        (*ok[:5], L["A"], L["B"].cpu()),                             # B on the host
    ]
    for args in bad_cases:
        with pytest.raises(ValueError):
            gpu_api.forward(*args)
    with pytest.raises(ValueError):
        gpu_api.forward(*ok, y=torch.empty((8, 32), device="cuda"))
    with pytest.raises(ValueError):
        gpu_api.backward(L["desc"], L["dy"][:, :32].contiguous(), *ok[1:])
    with pytest.raises(ValueError):
        gpu_api.backward(L["desc"], L["dy"], L["x"][:4].contiguous(), *ok[2:])
    with pytest.raises(ValueError):
        gpu_api.merge(L["desc"], L["g_beta"], L["A"], L["B"][:, :32].contiguous())


def test_streaming_status_word_stays_clear(gpu_api):
    """A few-token forward that completes leaves the workspace's status word as the caller set
    it (zero): the word is only written when a bounded wait for another block runs out."""
    cfg = synth.LayerConfig("stat", 4, 2048, 2048, 4, 32, 8, 0.5, seed=5)
    L = layer_on_gpu(gpu_api, cfg)
    ws = torch.zeros(gpu_api.workspace_bytes(L["desc"], 16, gpu_api.OP_FORWARD), dtype=torch.uint8, device="cuda")
    for T in (1, 4):
        gpu_api.forward(L["desc"], L["x"][:T].contiguous(), L["packed"], L["g_alpha"], L["g_beta"], ws=ws)
    assert gpu_api.streaming_status(ws) == 0


@pytest.mark.parametrize("layout", ["triple", "deployed", "factors16"])
def test_status_word_stays_clear_up_to_64_tokens(gpu_api, layout):
    """The same of the kernel for 33 to 64 tokens (deployed from 5), whose blocks wait for each other too: its
    flags and the word are where the few-token kernels have them, so one workspace serves both."""
    cfg = synth.LayerConfig("stat", 64, 4096, 4096, 4, 64, 8, 0.5, seed=6)
    L = layer_on_gpu(gpu_api, cfg)
    d, ab = L["desc"], (L["g_alpha"], L["g_beta"])
    op = gpu_api.OP_FORWARD_FACTORS16 if layout == "factors16" else gpu_api.OP_FORWARD
    ws = torch.zeros(gpu_api.workspace_bytes(d, 64, op), dtype=torch.uint8, device="cuda")
    dep = gpu_api.deploy(d, L["packed"], *ab)
    f16 = gpu_api.pack_factors16(d, *ab)
    for T in (64, 40, 4, 64):
        x = L["x"][:T].contiguous()
        if layout == "triple":
            gpu_api.forward(d, x, L["packed"], *ab, ws=ws)
        elif layout == "deployed":
            gpu_api.forward_deployed(d, x, dep, packed=L["packed"], ws=ws)
        else:
            gpu_api.forward_factors16(d, x, L["packed"], f16, ws=ws)
        assert gpu_api.streaming_status(ws) == 0, T
        flags = ws.view(torch.int64)[:256]
        assert int(flags.count_nonzero()) == 0, T   # every flag raised has been consumed


@pytest.mark.parametrize("w_std", [1e-5, 1e-7, 30.0])
def test_weights_far_from_unit_scale(gpu_api, w_std):
    """The dense path converts the factors to fp16 only after a power-of-two scale of its own
    (per output column forward, per call backward), so weights far below fp16's normal range
    -- or far above the usual 0.02 -- keep the same relative accuracy."""
    cfg = synth.LayerConfig("tiny_w", 300, 512, 264, 4, 32, 8, 0.5, seed=41, w_std=w_std, ab_std=0.02 * w_std / 0.02)
    L = layer_on_gpu(gpu_api, cfg)
    d = L["np"]
    w = (L["packed"], L["g_alpha"], L["g_beta"], L["A"], L["B"])
    y = gpu_api.forward(L["desc"], L["x"], *w)
    dx, dA, dB = gpu_api.backward(L["desc"], L["dy"], L["x"], *w)
    ref = oracle.forward(d["x"], L["codes"], L["alpha"], L["beta"], cfg.group, d["A"], d["B"], cfg.s)
    rdx, rdA, rdB = oracle.backward(d["dy"], d["x"], L["codes"], L["alpha"], L["beta"], cfg.group,
                                    d["A"], d["B"], cfg.s)
    errs = dict(y=rel_err(y.cpu().numpy(), ref), dx=rel_err(dx.cpu().numpy(), rdx),
                dA=rel_err(dA.cpu().numpy(), rdA), dB=rel_err(dB.cpu().numpy(), rdB))
    record(f"weights of std {w_std:g}", **errs)
    assert max(errs.values()) <= TOL, errs


def test_columns_of_very_different_scale(gpu_api):
    """Output columns whose weights differ by 2^40 in magnitude: the forward scales every
    column on its own, so each column is accurate relative to ITS largest output."""
    cfg = synth.LayerConfig("col_scales", 260, 256, 64, 4, 32, 0, 0.0, seed=43)
    d = synth.make_inputs(cfg)
    W = d["W"].copy()
    W[:, 1::2] *= np.float32(2.0 ** -40)
    codes, alpha, beta = oracle.quantize(W, 4, 32)
    L = layer_on_gpu(gpu_api, cfg, inputs=d, quantized=(codes, alpha, beta))
    y = gpu_api.forward(L["desc"], L["x"], L["packed"], L["g_alpha"], L["g_beta"]).cpu().numpy().astype(np.float64)
    ref = oracle.forward(d["x"], codes, alpha, beta, 32)
    per_col = np.abs(y - ref).max(axis=0) / np.abs(ref).max(axis=0)
    record("columns 2^40 apart", worst_column=float(per_col.max()))
    assert per_col.max() <= TOL


def test_imported_triples_far_from_the_mid_code(gpu_api):
    """Triples from another quantizer (through qalora_pack).  The dense path evaluates a weight
    as alpha (c - mid) + (beta + mid alpha) with the constant rounded to fp16, so its error per
    weight is bounded by 2^-11 |beta + mid alpha| (+ 2^-11 |alpha (c - mid)|) whatever codes the
    group uses -- stated in include/qalora.h.
    (a) zero-point groups alpha (c - z) with integer z anywhere in the code range, codes
        crowded at one end: the bound is a fraction of a quantization step, parity holds;
    (b) the degenerate encoding (codes 0, alpha = 1, beta = v): the error is bounded by
        2^-11 (|v| + 8), checked as such, not against the 2e-3 bar."""
    rng = np.random.default_rng(91)
    d_in, d_out, g, T = 512, 128, 32, 260
    x = torch.from_numpy(rng.standard_normal((T, d_in)).astype(np.float32)).to(torch.bfloat16)
    x64 = x.float().numpy().astype(np.float64)
    desc = gpu_api.make_desc(d_in, d_out, 4, g)
    # (a)
    z = rng.integers(0, 16, size=(d_in // g, d_out)).astype(np.float32)
    alpha = (rng.random((d_in // g, d_out), dtype=np.float32) * 0.01 + 0.002).astype(np.float32)
    lo = np.where(np.repeat(z, g, axis=0) < 8, 0, 12)
    codes = (lo + rng.integers(0, 4, size=(d_in, d_out))).astype(np.uint8)
    beta = oracle.beta_from_zero_point(alpha, z).astype(np.float32)
    y = gpu_api.forward(desc, x.cuda(), gpu_api.pack(desc, dev(codes)), dev(alpha), dev(beta))
    ref = oracle.forward(x64, codes, alpha, beta, g)
    err = rel_err(y.cpu().numpy(), ref)
    record("imported zero-point triples", y=err)
    assert err <= TOL
    # (b)
    v = (rng.standard_normal((d_in // g, d_out)) * 0.02).astype(np.float32)
    ones = np.ones_like(v)
    zeros = np.zeros((d_in, d_out), np.uint8)
    y = gpu_api.forward(desc, x.cuda(), gpu_api.pack(desc, dev(zeros)), dev(ones), dev(v))
    ref = oracle.forward(x64, zeros, ones, v, g)
    bound = 2.0 ** -11 * (np.abs(v).max() + 8.0) * np.abs(x64).sum(axis=1).max()
    assert np.abs(y.cpu().numpy() - ref).max() <= bound
