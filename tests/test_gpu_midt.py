"""The adapter-free forward between the few-token kernels and the dense one (up to 64 tokens): edges of its
token tiles, its slabs of 128 columns and its units of 512 rows, every code width and factor layout,
against the oracle, against the dense kernel and against itself.

Tolerance: operands are the dense kernel's (two fp16 factors per group and column and their fp16
combination, each rounded once: 3 * 2^-11 of the column's largest weight), whose bar of 2e-3 of the
largest output the other tests of that kernel use."""
import numpy as np
import pytest
import torch

import oracle
from paper_2309_14717_amd import synth
from helpers import layer_on_gpu, record, rel_err

pytestmark = pytest.mark.gpu


# `runs`: how the launch cuts the slabs of 128 columns -- whole slabs per block, every slab into the same number
# of parts (a hand-over each), or runs that end inside a slab and go on in the next.
@pytest.mark.parametrize("bits,group,d_in,d_out,tokens,runs", [
    (4, 32, 384, 640, 33, "whole"),      # one unit per slab, its fourth chunk absent
    (4, 32, 1024, 520, 48, "whole"),     # ragged last slab, two units per slab
    (4, 64, 640, 264, 49, "whole"),      # a unit of one chunk; two columns groups, the second nearly empty
    (4, 128, 4096, 1032, 64, "parts"),   # one group per chunk, a unit or two per part
    (4, 32, 2688, 4104, 64, "parts"),    # one unit per part
    (4, 32, 2048, 8200, 48, "parts"),    # the last part longer than the others
    (4, 128, 4096, 11008, 64, "cross"),
    (4, 64, 4096, 11016, 48, "cross"),
    (4, 32, 4096, 11016, 33, "cross"),
    (3, 32, 1152, 2056, 17, "parts"),
    (3, 64, 512, 136, 32, "whole"),
    (3, 128, 2048, 1160, 64, "parts"),
    (3, 64, 4096, 11016, 20, "cross"),
    (3, 32, 4096, 11016, 48, "cross"),
    (2, 32, 1024, 2048, 33, "whole"),
    (2, 64, 896, 72, 31, "whole"),
    (2, 128, 4224, 4096, 60, "parts"),
    (2, 32, 4096, 11016, 17, "cross"),
])
def test_mid_token_forward(gpu_api, bits, group, d_in, d_out, tokens, runs):
    units, slabs = -(-d_in // 512), -(-d_out // 128)
    blocks = gpu_api.mid_blocks(gpu_api.make_desc(d_in, d_out, bits, group), tokens)
    whole = blocks > 0 and (units == 1 or slabs % blocks == 0)
    assert ("dense" if blocks == 0 else "whole" if whole else "parts" if blocks % slabs == 0 else "cross") == runs
    cfg = synth.LayerConfig("mid", tokens + 64, d_in, d_out, bits, group, 8, 0.5, seed=71)
    L = layer_on_gpu(gpu_api, cfg)
    d, x = L["desc"], L["x"][:tokens].contiguous()
    # columns whose groups span twenty binades, growing and shrinking along the rows: the scale that
    # a column's accumulators carry has to follow
    alpha, beta = L["g_alpha"].clone(), L["g_beta"].clone()
    grow = torch.exp2(torch.linspace(-10, 10, alpha.shape[0], device=alpha.device))[:, None]
    for cols, f in ((slice(3, None, 8), grow), (slice(4, None, 8), grow.flip(0))):
        alpha[:, cols] *= f
        beta[:, cols] *= f
    ref = oracle.forward(L["np"]["x"][:tokens], L["codes"], alpha.cpu().numpy(), beta.cpu().numpy(), group)
    y = gpu_api.forward(d, x, L["packed"], alpha, beta)
    # the wide columns would hide the others: each column against its own largest output
    err = float(np.max(np.abs(y.cpu().numpy() - ref) / np.abs(ref).max(axis=0)))
    dense = gpu_api.forward(d, L["x"], L["packed"], alpha, beta)[:tokens]
    dense_err = float(np.max(np.abs(dense.cpu().numpy() - ref) / np.abs(ref).max(axis=0)))
    record(f"mid-token b={bits} g={group} {d_in}x{d_out} T={tokens}", y=err, dense=dense_err)
    assert err <= 2e-3
    assert float(((y - dense).abs().amax(0) / dense.abs().amax(0)).max()) <= 2e-3
    for _ in range(3):
        assert torch.equal(gpu_api.forward(d, x, L["packed"], alpha, beta), y)
    yb = gpu_api.forward(d, x, L["packed"], alpha, beta, out_dtype=torch.bfloat16)
    assert torch.equal(yb, y.to(torch.bfloat16))
    if bits == 4:
        dep = gpu_api.deploy(d, L["packed"], alpha, beta)
        assert torch.equal(gpu_api.forward_deployed(d, x, dep, packed=L["packed"]), y)
    f16 = gpu_api.pack_factors16(d, alpha, beta)
    same = gpu_api.forward(d, x, L["packed"], alpha.half().float(), beta.half().float())
    assert torch.equal(gpu_api.forward_factors16(d, x, L["packed"], f16), same)


@pytest.mark.parametrize("layout", ["triple", "deployed"])
def test_small_groups_beside_large_ones(gpu_api, layout):
    """Groups 2^22 below the largest of their column, multiplied by activations that are zero elsewhere: their
    fp16 factors must stay normal numbers, as they do on the dense kernel (a column's bound is brought to
    [2^13, 2^14), alpha is a sixteenth of it or more and 2^-14 the smallest normal number).  With a scale
    four binades lower the error is four times the dense kernel's."""
    g, d_in, d_out, T = 32, 1024, 1024, 40
    cfg = synth.LayerConfig("small", 2 * T, d_in, d_out, 4, g, 8, 0.5, seed=73)
    L = layer_on_gpu(gpu_api, cfg)
    groups = torch.arange(d_in // g, device="cuda") % 4     # of every chunk the first group is the large one
    f = torch.where(groups == 0, 1.0, 2.0 ** -22)[:, None]
    alpha, beta = L["g_alpha"] * f, L["g_beta"] * f
    x = torch.where(groups.repeat_interleave(g) == 0, torch.zeros((), device="cuda"), L["x"].float()).to(torch.bfloat16)
    xt = x[:T].contiguous()
    if layout == "deployed":
        y = gpu_api.forward_deployed(L["desc"], xt, gpu_api.deploy(L["desc"], L["packed"], alpha, beta), packed=L["packed"])
    else:
        y = gpu_api.forward(L["desc"], xt, L["packed"], alpha, beta)
    ref = oracle.forward(xt.float().cpu().numpy(), L["codes"], alpha.cpu().numpy(), beta.cpu().numpy(), g)
    err = float(np.max(np.abs(y.cpu().numpy() - ref) / np.abs(ref).max(axis=0)))
    dense = gpu_api.forward(L["desc"], x, L["packed"], alpha, beta)[:T]
    dense_err = float(np.max(np.abs(dense.cpu().numpy() - ref) / np.abs(ref).max(axis=0)))
    record(f"small groups, {layout}", y=err, dense=dense_err)
    assert dense_err <= 2e-3 and err <= 1.5 * dense_err


def test_mid_token_forward_non_finite(gpu_api):
    """Infinities and NaN in a group reach the outputs of that column and no other."""
    cfg = synth.LayerConfig("mid_nan", 40, 1024, 520, 4, 32, 8, 0.5, seed=72)
    L = layer_on_gpu(gpu_api, cfg)
    alpha, beta = L["g_alpha"].clone(), L["g_beta"].clone()
    y0 = gpu_api.forward(L["desc"], L["x"], L["packed"], alpha, beta)
    alpha[5, 17], beta[31, 300], beta[0, 519] = float("nan"), float("inf"), float("-inf")
    y = gpu_api.forward(L["desc"], L["x"], L["packed"], alpha, beta)
    hit = [17, 300, 519]
    assert not torch.isfinite(y[:, hit]).any()
    keep = [j for j in range(520) if j not in hit]
    assert torch.equal(y[:, keep], y0[:, keep])
