"""The adapter's gradients at the edges of their launches.  By way of Z = pool(x)^T dy: one launch (up to 640 tokens and
256 blocks of 128 groups x 32 columns) or runs of (tile, 64 tokens) units whose partial sums meet, more than 128
groups (dB in shares), group counts that are no multiple of eight, ranks beside multiples of sixteen; against
the oracle.  By way of U = pool(x) A and dU = dy B^T, further below.  Tolerance: the operands hold all bits of theirs (pool(x) as three bf16 pieces); every sum is one of fp32
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


SHAPES = [
    (1, 128, 8, 4, 32, 1),          # one token, a quarter of a column block
    (63, 1024, 1000, 4, 8, 17),     # 128 groups exactly; rank beside a multiple of 16
    (65, 1032, 264, 4, 8, 128),     # 129 groups: a second share of one group
    (640, 4160, 40, 2, 32, 15),     # the longest batch in one launch; two shares, 130 groups
    (641, 416, 520, 4, 32, 16),     # the first in two; 13 groups
    (700, 2080, 1032, 4, 8, 33),    # 260 groups: three tiles of them, runs that cross tiles
    (1000, 96, 8200, 3, 32, 64),    # three groups; more tiles than a run's
    (130, 1024, 8256, 4, 8, 8),     # 258 blocks: two launches at few tokens (by U: the rank is low)
    (130, 1024, 8256, 4, 8, 100),   # ... by Z
    (4096, 256, 136, 4, 128, 64),   # two groups, two tiles of columns, 64 steps
    (65, 1920, 264, 4, 32, 24),     # 60 groups: tiles of 64
    (700, 1920, 520, 4, 32, 24),    # ... in two launches
    (650, 2208, 200, 4, 32, 100),   # 69 groups: the tile's third quarter begins; columns end inside the second tile
    (705, 3104, 136, 2, 32, 40),    # 97 groups: its last quarter begins
    (5, 4800, 64, 4, 40, 8),        # rows pooled by a block each in the forward, groups beside powers of two
    (200, 4128, 64, 4, 32, 8),      # ... and beyond a wavefront's registers; 129 groups
]
# by way of U and dU: (tokens, d_in, d_out, group, ((columns, rank) of each part))
BY_U = [
    (130, 1032, 8256, 8, ((8256, 17),)),                   # 129 groups, a second tile of one; rank beside a multiple of 16
    (1, 4136, 5000, 8, ((5000, 33),)),                     # one token; 517 groups
    (65, 3080, 6152, 8, ((6152, 100),)),                   # a token in the second block; columns beside a step
    (1025, 3080, 2056, 8, ((2056, 8),)),                   # blocks of 256 tokens, one of one; rank of one chunk
    (1300, 13824, 4096, 32, ((4096, 128),)),               # ... with the largest rank; several steps a share of dA
    (700, 4128, 6176, 16, ((2080, 40), (32, 128), (4064, 8))),   # parts: widths beside steps and tiles, three ranks
]


@pytest.mark.parametrize("tokens,d_in,d_out,bits,group,rank", SHAPES)
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


@pytest.mark.parametrize("tokens,d_in,d_out,group,parts", BY_U)
def test_gradients_by_way_of_u(gpu_api, tokens, d_in, d_out, group, parts):
    """Against the same products in 64 bits, from x and from the kept activations, added to what is there."""
    api, gen, L, s = gpu_api, torch.Generator("cuda").manual_seed(94), d_in // group, 0.5
    rand = lambda *n: torch.randn(n, device="cuda", generator=gen)   # noqa: E731
    desc = api.make_desc(d_in, d_out, 4, group, 0 if len(parts) > 1 else parts[0][1], s)
    w = api.quantize(desc, rand(d_in, d_out))
    x, dy = rand(tokens, d_in).bfloat16(), rand(tokens, d_out).bfloat16()
    ads = [(rand(L, r), rand(r, n), s) for n, r in parts]
    if len(parts) > 1:
        kept = api.forward_shared(desc, x, *w, ads, keep=True)[1]
        grads = [[(torch.ones_like(A), torch.ones_like(B)) for A, B, _ in ads] for _ in range(2)]
        api.backward_shared(desc, dy, x, None, *w, ads, grads=grads[0])
        api.backward_shared(desc, dy, None, kept, *w, ads, grads=grads[1], accumulate=True)
    else:
        A, B, _ = ads[0]
        kept = api.forward_keep(desc, x, *w, A, B)[1]
        grads = [[api.backward(desc, dy, x, *w, A, B)[1:]],
                 [api.backward_kept(desc, dy, kept, *w, A, B, dA=torch.ones_like(A), dB=torch.ones_like(B),
                                    accumulate=True)[1:]]]
    P, col = x.double().view(tokens, L, group).mean(2), 0
    for (n, r), (A, B, _), got, added in zip(parts, ads, *grads):
        y = dy[:, col:col + n].double()
        ref = (s * P.T @ (y @ B.double().T), s * (P @ A.double()).T @ y)
        errs = [rel_err(g.cpu().numpy(), t.cpu().numpy()) for g, t in zip(got, ref)]
        record(f"gradients by U T={tokens} L={L} {n} r={r}", dA=errs[0], dB=errs[1])
        assert max(errs) <= TOL_SUMS
        assert all(torch.equal(b, 1 + a) for a, b in zip(got, added))
        col += n


def test_values_that_are_not_finite_by_way_of_u(gpu_api):
    """As above: an infinity in x, in dy, and in a column of dy that belongs to another part."""
    api, gen, L = gpu_api, torch.Generator("cuda").manual_seed(95), 258
    rand = lambda *n: torch.randn(n, device="cuda", generator=gen)   # noqa: E731
    desc = api.make_desc(8 * L, 5024, 4, 8)
    w = api.quantize(desc, rand(8 * L, 5024))
    ads = [(rand(L, r), rand(r, n), 0.5) for n, r in ((2496, 20), (2528, 40))]

    def bad(x, dy):
        grads = [(torch.zeros_like(A), torch.zeros_like(B)) for A, B, _ in ads]
        api.backward_shared(desc, dy, x, None, *w, ads, grads=grads)
        return [~torch.isfinite(t).cpu().numpy() for pair in grads for t in pair]

    x, dy = rand(70, 8 * L).bfloat16(), rand(70, 5024).bfloat16()
    xi, yi = x.clone(), dy.clone()
    xi[3, 40], yi[5, 2495] = float("inf"), float("inf")
    dA0, dB0, dA1, dB1 = bad(xi, dy)
    for dA in (dA0, dA1):
        assert dA[5].all() and not np.delete(dA, 5, axis=0).any()
    dA0, dB0, dA1, dB1 = bad(x, yi)
    assert dA0.all() and not dA1.any() and not dB1.any()
    assert dB0[:, 2495].all() and not np.delete(dB0, 2495, axis=1).any()
