"""The backward's conversion of long dy rows by a whole block: rows just above what one wavefront takes, at
the edges of the block's register batches (16384 and 32768 elements) and beyond them, the largest
value in the row's last piece (a missed piece would let the fp16 copy overflow).  dx against the
oracle at the bar of the dense product (2e-3 of the largest value)."""
import pytest
import torch

import oracle
from paper_2309_14717_amd import synth
from helpers import layer_on_gpu, record, rel_err

pytestmark = pytest.mark.gpu


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
