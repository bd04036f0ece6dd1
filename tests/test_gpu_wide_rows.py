"""The backward's conversion of long dy rows by a whole block: rows just above what one wavefront takes, at
the edges of the block's register batches (16384 and 32768 elements) and beyond them, the largest
value in the row's last piece (a missed piece would let the fp16 copy overflow).  dx against the
oracle at the bar of the dense product (2e-3 of the largest value).  The forward's rows beside its factor job, by
a block or a wavefront each, on either side of where the rule changes (checked on the host), at the same bar."""
import pytest
import torch


import oracle
from paper_2309_14717_amd import synth
from helpers import layer_on_gpu, record, rel_err
from host_code import host_library


@pytest.mark.gpu
@pytest.mark.parametrize("d_out", [4104, 16384, 16392, 22016, 32768, 32776])
@pytest.mark.parametrize("tokens", [3, 130, 520])
def test_long_gradient_rows(gpu_api, tokens, d_out):
    cfg = synth.LayerConfig("wide", tokens, 128, d_out, 4, 32, 8, 0.5, seed=91)
    L = layer_on_gpu(gpu_api, cfg)
    n = L["np"]
    dy = L["dy"].clone()
    dy[::2, -1] *= 4096.0
    dy[1::2, 0] *= 4096.0
    rdx, rdA, rdB = oracle.backward(dy.float().cpu().numpy(), n["x"], L["codes"], L["alpha"], L["beta"], 32,
                                    n["A"], n["B"], cfg.s)
    dx, dA, dB = gpu_api.backward(L["desc"], dy, L["x"], L["packed"], L["g_alpha"], L["g_beta"], L["A"], L["B"])
    err = rel_err(dx.float().cpu().numpy(), rdx)
    record(f"long dy rows T={tokens} d_out={d_out}", dx=err)
    assert err <= 2e-3
    assert rel_err(dA.cpu().numpy(), rdA) <= 2e-3 and rel_err(dB.cpu().numpy(), rdB) <= 2e-3


#    tokens d_in d_out group rank pooled  by a block
ROWS = [
    (256, 512, 256, 32, 0, False, True),
    (257, 512, 256, 32, 0, False, False),
    (64, 4128, 256, 32, 0, False, True),        # more than a wavefront takes in one sweep, small groups
    (65, 4128, 256, 32, 0, False, False),
    (97, 4160, 264, 64, 0, False, True),        # ... larger ones
    (256, 512, 264, 32, 8, False, True),        # an adapter to fold, nothing kept
    (257, 512, 264, 32, 8, False, False),
    (100, 512, 264, 32, 104, False, False),     # ... of a high rank
    (511, 4224, 8208, 32, 40, True, True),      # 513 blocks of the job
    (512, 4224, 8208, 32, 40, True, False),     # ... and as many of rows before its last one: more than run at once
    (520, 4224, 8208, 64, 8, True, True),       # ... where the job's are short
    (200, 4224, 264, 32, 48, False, False),     # long rows, a long job
    (200, 4224, 264, 32, 48, True, True),       # ... that take as long with pooling
    (200, 13824, 13824, 32, 128, True, False),
]


def test_rows_by_block_or_wavefront(tmp_path):
    lib = host_library(tmp_path, "front_plan", """
#include "front_plan.hpp"
extern "C" int by_block(int T, int d_in, int g, int d_out, int fold, int rank, int pooled) {
  return qalora::front_rows_by_block(T, d_in, g, d_out, fold, rank, pooled);
}
""")
    for tokens, d_in, d_out, group, rank, pooled, by_block in ROWS:
        assert bool(lib.by_block(tokens, d_in, group, d_out, rank > 0, rank, pooled)) == by_block, (tokens, d_in, d_out, group, rank)
    # measured: 10 to 16 % longer by wavefronts
    assert lib.by_block(300, 13824, 128, 5120, 0, 0, 0) and lib.by_block(200, 22016, 128, 8192, 0, 0, 0)
    assert lib.by_block(200, 13824, 128, 13824, 1, 16, 1) and lib.by_block(500, 13824, 128, 5120, 1, 16, 0)


@pytest.mark.gpu
@pytest.mark.parametrize("tokens,d_in,d_out,group,rank,pooled,by_block", ROWS[:-1])
def test_forward_rows(gpu_api, tokens, d_in, d_out, group, rank, pooled, by_block):
    api, gen, L = gpu_api, torch.Generator("cuda").manual_seed(96), d_in // group
    rand = lambda *n: torch.randn(n, device="cuda", generator=gen)   # noqa: E731
    desc = api.make_desc(d_in, d_out, 4, group, rank, 0.5)
    packed, alpha, beta = api.quantize(desc, rand(d_in, d_out))
    x = rand(tokens, d_in)
    x[::2, -1] *= 4096.0
    x[1::2, 0] *= 4096.0
    x = x.bfloat16()
    rows = lambda t: t.double().repeat_interleave(group, 0)   # noqa: E731
    ref = x.double() @ (api.unpack(desc, packed).double() * rows(alpha) + rows(beta))
    ad = (rand(L, rank), rand(rank, d_out)) if rank else (None, None)
    if rank:
        ref += 0.5 * (x.double().view(tokens, L, group).mean(2) @ ad[0].double()) @ ad[1].double()
    if pooled:
        y, kept = api.forward_keep(desc, x, packed, alpha, beta, *ad)
        dy = rand(tokens, d_out).bfloat16()
        a, b = (api.backward(desc, dy, x, packed, alpha, beta, *ad), api.backward_kept(desc, dy, kept, packed, alpha, beta, *ad))
        errs = [rel_err(s.cpu().numpy(), t.cpu().numpy()) for s, t in zip(a[1:], b[1:])]   # pooled by blocks and by wavefronts
        assert max(errs) <= 1e-5
    else:
        y = api.forward(desc, x, packed, alpha, beta, *ad)
    err = rel_err(y.cpu().numpy(), ref.cpu().numpy())
    record(f"forward rows T={tokens} {d_in}x{d_out} g={group} r={rank}", y=err)
    assert err <= 2e-3
