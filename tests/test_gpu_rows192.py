"""The dense contraction on 192-row tiles, where they save padding or a round of blocks: forward and both
gradients at the edges of the tile, and where its last tile ends past the rows the fp16 copies are
padded to (200 rows: tiles to 384, copies to 256), against the oracle.  Tolerances: those of the
256-row tile in the other tests (forward and dx 2e-3 of the largest value; the operands are the
same fp16 numbers, summed in the same order)."""
import pytest
import torch

import oracle
from paper_2309_14717_amd import synth
from helpers import layer_on_gpu, record, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits,group,tokens,d_in,d_out", [
    (4, 32, 129, 512, 520),    # one tile, mostly padding
    (4, 64, 192, 768, 256),    # one whole tile
    (3, 32, 193, 512, 520),    # a second tile of one row
    (4, 32, 200, 512, 520),    # tiles end 128 rows past the copies
    (2, 32, 960, 320, 520),    # five whole tiles, 64 rows short of the copies
    (2, 32, 384, 320, 1032),   # two whole tiles
    (3, 64, 320, 640, 776),
    (4, 32, 600, 256, 22016),  # 256-row tiles leave a ragged round: 258 blocks
    (2, 64, 560, 512, 136),
])
def test_rows192(gpu_api, bits, group, tokens, d_in, d_out):
    cfg = synth.LayerConfig("r192", tokens, d_in, d_out, bits, group, 8, 0.5, seed=81)
    L = layer_on_gpu(gpu_api, cfg)
    d, n = L["desc"], L["np"]
    A, B = n["A"], n["B"]
    y = gpu_api.forward(d, L["x"], L["packed"], L["g_alpha"], L["g_beta"], L["A"], L["B"])
    ref = oracle.forward(n["x"], L["codes"], L["alpha"], L["beta"], group, A, B, cfg.s)
    ey = rel_err(y.cpu().numpy(), ref)
    dx, dA, dB = gpu_api.backward(d, L["dy"], L["x"], L["packed"], L["g_alpha"], L["g_beta"], L["A"], L["B"])
    rdx, rdA, rdB = oracle.backward(n["dy"], n["x"], L["codes"], L["alpha"], L["beta"], group, A, B, cfg.s)
    ex = rel_err(dx.float().cpu().numpy(), rdx)
    record(f"192-row tile b={bits} T={tokens} {d_in}x{d_out}", y=ey, dx=ex)
    assert ey <= 2e-3 and ex <= 2e-3
    assert rel_err(dA.cpu().numpy(), rdA) <= 2e-3 and rel_err(dB.cpu().numpy(), rdB) <= 2e-3
    assert torch.equal(gpu_api.forward(d, L["x"], L["packed"], L["g_alpha"], L["g_beta"], L["A"], L["B"]), y)
