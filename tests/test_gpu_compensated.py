"""Error-compensated code selection on the GPU (qalora_quantize_compensated) against the oracle:
the operation order is part of the definition, so codes, alpha and beta must agree bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2309_14717_amd import synth
from helpers import dev
from test_oracle_compensated import hessian, hessian_error

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits,g,d_in,d_out", [(4, 32, 384, 40), (3, 64, 256, 16), (2, 128, 512, 72), (4, 16, 208, 24)])
def test_compensated_bit_exact(gpu_api, bits, g, d_in, d_out):
    W = synth.make_inputs(synth.LayerConfig("t", 1, d_in, d_out, bits, g, 1, seed=40 + bits), want=("W",))["W"]
    H, U = hessian(d_in, 4 * d_in, seed=bits)
    U32 = np.ascontiguousarray(U.astype(np.float32))
    desc = gpu_api.make_desc(d_in, d_out, bits, g)
    if gpu_api.check_desc(desc) != gpu_api.OK:
        pytest.skip("group size outside the packed format for this code width")
    packed, alpha, beta = gpu_api.quantize_compensated(desc, dev(W), dev(U32))
    codes = gpu_api.unpack(desc, packed).cpu().numpy()
    c, a, b = oracle.quantize_compensated(W, U32, bits, g, block=128)
    assert np.array_equal(codes, c)
    assert np.array_equal(alpha.cpu().numpy().view(np.uint32), a.view(np.uint32))
    assert np.array_equal(beta.cpu().numpy().view(np.uint32), b.view(np.uint32))
    # and it does what it is for: less output error under H than plain rounding
    e_rtn = hessian_error(W, *oracle.quantize(W, bits, g), g, H)
    assert hessian_error(W, codes, a, b, g, H) < e_rtn


@pytest.mark.parametrize("bits,g,d_in,d_out,w_exp,u_exp,kind", [
    (4, 8, 136, 8, 0, 0, "plain"),       # a panel and half a tile; groups inside a tile; half a column block
    (4, 8, 8, 16, 0, 0, "plain"),
    (4, 32, 64, 24, 0, 0, "plain"),      # one panel, not a whole one
    (4, 8, 120, 40, 0, 0, "plain"),
    (3, 32, 96, 16, 0, 0, "plain"),
    (4, 8, 264, 24, 0, 0, "plain"),      # half a tile in the last of three panels
    (4, 128, 256, 24, 0, 0, "plain"),    # a group per panel
    (3, 32, 416, 40, 0, 0, "plain"),     # high-bit words of a ragged last panel
    (2, 16, 144, 56, 0, 0, "plain"),
    (4, 32, 384, 24, -70, 0, "plain"),   # operands outside the reciprocals' range: real divisions
    (4, 32, 384, 24, 70, 0, "plain"),
    (4, 32, 256, 24, 0, -50, "plain"),
    (4, 32, 256, 24, 0, 50, "plain"),
    (4, 32, 256, 24, 0, 0, "zeros"),     # groups of signed zeros
    (4, 8, 256, 24, 0, 0, "pruned"),     # minima that are signed zeros
    (4, 16, 256, 48, 0, 0, "columns"),   # safe and unsafe columns side by side
    (3, 32, 384, 40, 0, 0, "tiny"),      # single elements far below the rest
])
def test_compensated_edges(gpu_api, bits, g, d_in, d_out, w_exp, u_exp, kind):
    r = np.random.RandomState(d_in + d_out + bits)
    W = (r.randn(d_in, d_out) * 0.02).astype(np.float32) * np.float32(2.0 ** w_exp)
    if kind == "zeros":
        W = np.where(r.rand(d_in, d_out) < 0.5, np.float32(-0.0), np.float32(0.0))
    elif kind == "pruned":
        W = np.maximum(W, 0) * np.where(r.rand(d_in, d_out) < 0.5, 1, -0.0).astype(np.float32)
    elif kind == "columns":
        W *= np.float32(2.0) ** r.randint(-140, 100, size=(1, d_out)).astype(np.float32)
    elif kind == "tiny":
        W[r.rand(d_in, d_out) < 0.1] *= np.float32(1e-36)
    _, U = hessian(d_in, 2 * d_in, seed=3)
    U32 = np.ascontiguousarray((U * 2.0 ** u_exp).astype(np.float32))
    desc = gpu_api.make_desc(d_in, d_out, bits, g)
    packed, alpha, beta = gpu_api.quantize_compensated(desc, dev(W), dev(U32))
    c, a, b = oracle.quantize_compensated(W, U32, bits, g, block=128)
    assert np.array_equal(gpu_api.unpack(desc, packed).cpu().numpy(), c)
    assert np.array_equal(alpha.cpu().numpy().view(np.uint32), a.view(np.uint32))
    assert np.array_equal(beta.cpu().numpy().view(np.uint32), b.view(np.uint32))


@pytest.mark.parametrize("bits,g", [(4, 8), (4, 16), (4, 32), (3, 64), (2, 128)])
def test_compensated_non_finite_weights(gpu_api, bits, g):
    """A NaN or an infinity spoils its column from its row on, in the group's factors too where Eq. 1's running
    minimum and maximum meet it first; the other columns keep their bits."""
    d_in, d_out = 384, 40
    r = np.random.RandomState(g)
    W = (r.randn(d_in, d_out) * 0.02).astype(np.float32)
    for k, v in enumerate((np.nan, np.inf, -np.inf)):
        W[g, 3 + k] = v                 # first row of a group
        W[128 + g // 2, 13 + k] = v     # inside a group
        W[0, 23 + k] = v
    _, U = hessian(d_in, 2 * d_in, seed=4)
    U32 = np.ascontiguousarray(U.astype(np.float32))
    desc = gpu_api.make_desc(d_in, d_out, bits, g)
    packed, alpha, beta = gpu_api.quantize_compensated(desc, dev(W), dev(U32))
    c, a, b = oracle.quantize_compensated(W, U32, bits, g, block=128)
    assert np.array_equal(alpha.cpu().numpy(), a, equal_nan=True)
    assert np.array_equal(beta.cpu().numpy(), b, equal_nan=True)
    clean = np.isfinite(W).all(axis=0)
    assert clean.sum() == d_out - 9
    assert np.array_equal(gpu_api.unpack(desc, packed).cpu().numpy()[:, clean], c[:, clean])


def test_compensated_many_blocks_and_rerun(gpu_api):
    """A layer of sixteen lazy row blocks and 128 column blocks (all compute units busy, two
    block generations), bit for bit against the oracle, and twice: the row lanes of a column
    live in different wavefronts, so an ordering mistake between them would show as a result
    that differs between runs or from the oracle."""
    bits, g, d_in, d_out = 4, 32, 2048, 2048
    W = synth.make_inputs(synth.LayerConfig("t", 1, d_in, d_out, bits, g, 1, seed=61), want=("W",))["W"]
    _, U = hessian(d_in, 2 * d_in, seed=9)
    U32 = np.ascontiguousarray(U.astype(np.float32))
    desc = gpu_api.make_desc(d_in, d_out, bits, g)
    Wd, Ud = dev(W), dev(U32)
    p1, a1, b1 = gpu_api.quantize_compensated(desc, Wd, Ud)
    p2, a2, b2 = gpu_api.quantize_compensated(desc, Wd, Ud)
    assert torch.equal(p1, p2) and torch.equal(a1, a2) and torch.equal(b1, b2)
    c, a, b = oracle.quantize_compensated(W, U32, bits, g, block=128)
    assert np.array_equal(gpu_api.unpack(desc, p1).cpu().numpy(), c)
    assert np.array_equal(a1.cpu().numpy().view(np.uint32), a.view(np.uint32))
    assert np.array_equal(b1.cpu().numpy().view(np.uint32), b.view(np.uint32))


def test_compensated_identity_is_plain_quantize(gpu_api):
    d_in, d_out = 256, 64
    W = synth.make_inputs(synth.LayerConfig("t", 1, d_in, d_out, 4, 32, 1, seed=50), want=("W",))["W"]
    desc = gpu_api.make_desc(d_in, d_out, 4, 32)
    p1, a1, b1 = gpu_api.quantize_compensated(desc, dev(W), torch.eye(d_in, device="cuda"))
    p0, a0, b0 = gpu_api.quantize(desc, dev(W))
    assert torch.equal(p1, p0) and torch.equal(a1, a0) and torch.equal(b1, b0)


def test_compensated_layer_runs_on_the_result(gpu_api):
    """The triple feeds the layer like any other: forward parity against the oracle on it."""
    d_in, d_out, T = 512, 128, 33
    cfg = synth.LayerConfig("t", T, d_in, d_out, 4, 32, 8, 0.5, seed=51)
    d = synth.make_inputs(cfg)
    _, U = hessian(d_in, 2048, seed=6)
    U32 = np.ascontiguousarray(U.astype(np.float32))
    desc = gpu_api.make_desc(d_in, d_out, 4, 32, 8, 0.5)
    packed, alpha, beta = gpu_api.quantize_compensated(desc, dev(d["W"]), dev(U32))
    c, a, b = oracle.quantize_compensated(d["W"], U32, 4, 32)
    y = gpu_api.forward(desc, dev(d["x"], torch.bfloat16), packed, alpha, beta, dev(d["A"]), dev(d["B"]))
    ref = oracle.forward(d["x"], c, a, b, 32, d["A"], d["B"], 0.5)
    assert np.abs(y.cpu().numpy() - ref).max() <= 2e-3 * np.abs(ref).max()


def test_compensated_rejects_groups_that_straddle_blocks(gpu_api):
    desc = gpu_api.make_desc(384, 64, 4, 96)
    with pytest.raises(gpu_api.QaloraError) as e:
        gpu_api.quantize_compensated(desc, torch.zeros(384, 64, device="cuda"), torch.eye(384, device="cuda"))
    assert e.value.status == gpu_api.EUNSUPPORTED
