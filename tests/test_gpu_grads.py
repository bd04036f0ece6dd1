"""The adapter's gradients by way of Z = pool(x)^T dy, at the edges of its launches: one launch (up to 640 tokens and
256 blocks of 128 groups x 32 columns) or runs of (tile, 64 tokens) units whose partial sums meet, more than 128
groups (dB in shares), group counts that are no multiple of eight, ranks beside multiples of sixteen.  Against
the oracle.  Tolerance: the operands hold all bits of theirs (pool(x) as three bf16 pieces); every sum is one of fp32
rounding errors, 2^-24 of the sums on the way, whose signs add up like sqrt(terms): 2^-24 sqrt(4096 + 8256) < 7e-6 of
the largest, with room for sums on the way that are larger than their end."""
import numpy as np
import pytest
import torch

import oracle
from helpers import layer_on_gpu, record, rel_err
from paper_2309_14717_amd import synth

pytestmark = pytest.mark.gpu

# (the bound above, four times)
TOL_SUMS = 2.8e-5


@pytest.mark.parametrize("tokens,d_in,d_out,bits,group,rank", [
    (1, 128, 8, 4, 32, 1),          # one token, a quarter of a column block
    (63, 1024, 1000, 4, 8, 17),     # 128 groups exactly; rank beside a multiple of 16
    (65, 1032, 264, 4, 8, 128),     # 129 groups: a second share of one group
    (640, 4160, 40, 2, 32, 15),     # the longest batch in one launch; two shares, 130 groups
    (641, 416, 520, 4, 32, 16),     # the first in two; 13 groups
    (700, 2080, 1032, 4, 8, 33),    # 260 groups: three tiles of them, runs that cross tiles
    (1000, 96, 8200, 3, 32, 64),    # three groups; more tiles than a run's
    (130, 1024, 8256, 4, 8, 8),     # 258 blocks: two launches at few tokens
    (4096, 256, 136, 4, 128, 64),   # two groups, two tiles of columns, 64 steps
    (5, 4800, 64, 4, 40, 8),        # rows pooled by a block each in the forward, groups beside powers of two
    (200, 4128, 64, 4, 32, 8),      # ... and beyond a wavefront's registers; 129 groups
])
def test_gradients(gpu_api, tokens, d_in, d_out, bits, group, rank):
    cfg = synth.LayerConfig("grads", tokens, d_in, d_out, bits, group, rank, 0.5, seed=91)
    L = layer_on_gpu(gpu_api, cfg)
    d, n = L["desc"], L["np"]
    w = (L["packed"], L["g_alpha"], L["g_beta"], L["A"], L["B"])
    _, rdA, rdB = oracle.backward(n["dy"], n["x"], L["codes"], L["alpha"], L["beta"], group, n["A"], n["B"], cfg.s)
    dx, dA, dB = gpu_api.backward(d, L["dy"], L["x"], *w)
    eA, eB = rel_err(dA.cpu().numpy(), rdA), rel_err(dB.cpu().numpy(), rdB)
    record(f"gradients T={tokens} {d_in}x{d_out} g={group} r={rank}", dA=eA, dB=eB)
    assert eA <= TOL_SUMS and eB <= TOL_SUMS
    # from the kept activations, added to what is there: the same sums
    _, kept = gpu_api.forward_keep(d, L["x"], *w)
    a0, b0 = torch.ones_like(dA), torch.full_like(dB, -2.0)
    kdx, kA, kB = gpu_api.backward_kept(d, L["dy"], kept, *w, dA=a0.clone(), dB=b0.clone(), accumulate=True)
    assert torch.equal(kdx, dx)
    assert torch.equal(kA, a0 + dA) and torch.equal(kB, b0 + dB)
    again = gpu_api.backward(d, L["dy"], L["x"], *w)
    assert torch.equal(again[1], dA) and torch.equal(again[2], dB)


def test_values_that_are_not_finite_stay_in_their_groups_and_columns(gpu_api):
    """An infinity in x reaches its group's row of dA, one in dy its column of dB."""
    cfg = synth.LayerConfig("grads", 70, 512, 256, 4, 32, 16, 0.5, seed=92)
    L = layer_on_gpu(gpu_api, cfg)
    w = (L["packed"], L["g_alpha"], L["g_beta"], L["A"], L["B"])
    x, dy = L["x"].clone(), L["dy"].clone()
    x[3, 40] = float("inf")
    _, dA, _ = gpu_api.backward(L["desc"], dy, x, *w)
    bad = ~torch.isfinite(dA).cpu().numpy()
    assert bad[1].all() and not np.delete(bad, 1, axis=0).any()
    dy[5, 77] = float("inf")
    _, _, dB = gpu_api.backward(L["desc"], dy, L["x"], *w)
    bad = ~torch.isfinite(dB).cpu().numpy()
    assert bad[:, 77].all() and not np.delete(bad, 77, axis=1).any()


@pytest.mark.parametrize("tokens,d_in,d_out,group,rank", [(1, 1024, 1024, 32, 16), (700, 1024, 1024, 32, 16),
                                                          (700, 5120, 1032, 32, 8)])
def test_pooled_activations_keep_their_bits(gpu_api, tokens, d_in, d_out, group, rank):
    """One token that counts and one-hot adapters: every gradient is one product of a pooled activation and an element
    of dy.  The pooled activations need all their 24 bits, and no sum on the way to one rounds; the product is then
    within a few 2^-24 of the exact one.  (Two bf16 pieces leave up to 2^-18, rounding to one 2^-9.)"""
    api, gen, L = gpu_api, torch.Generator("cuda").manual_seed(93), d_in // group
    t = tokens // 2
    desc = api.make_desc(d_in, d_out, 4, group, rank, 1.0)
    w = api.quantize(desc, torch.randn(d_in, d_out, device="cuda", generator=gen))
    x, dy = torch.zeros(tokens, d_in, device="cuda"), torch.randn(tokens, d_out, device="cuda", generator=gen)
    for i, e in enumerate((-7, -15, -23)):   # eight bits each, one below the other
        x[t, i::group] = torch.randint(128, 200, (L,), device="cuda", generator=gen).float() * 2.0 ** e
    x, dy = x.bfloat16(), dy.bfloat16()
    ls, js = (torch.randperm(n, generator=gen, device="cuda")[:rank] for n in (L, d_out))
    A, B = torch.zeros(L, rank, device="cuda"), torch.zeros(rank, d_out, device="cuda")
    k = torch.arange(rank, device="cuda")
    A[ls, k], B[k, js] = 1.0, 1.0
    P = x[t].double().view(L, group).mean(1)
    assert torch.equal(P.float().double(), P)
    _, dA, dB = api.backward(desc, dy, x, *w, A, B)
    _, kept = api.forward_keep(desc, x, *w, A, B)
    _, kA, kB = api.backward_kept(desc, dy, kept, *w, A, B)
    for got, ref in ((dA, P[:, None] * dy[t].double()[js][None]), (dB, P[ls][:, None] * dy[t].double()[None])):
        assert ((got.double() - ref).abs() <= 2.0 ** -22 * ref.abs()).all()
    assert torch.equal(kA, dA) and torch.equal(kB, dB)
