"""Tile rows and K split of the dense product: what the rule gives at the edges of its range (host), and the
forward and both gradients on those launches against the oracle (gpu).  Tolerance: forward and dx 2e-3 of the
largest value, as for every other tile: the operands are the same fp16 numbers, only the order of the fp32
sums differs."""
import ctypes
import random

import pytest

import oracle
from helpers import layer_on_gpu, record, rel_err
from host_code import host_library
from paper_2309_14717_amd import api, synth

#        bits group tokens d_in d_out  forward's and backward's (tile rows, slices)
SHAPES = [
    (4, 32, 65, 1024, 1032, (64, 4), (64, 6)),       # one row in the second tile; backward: K = 1032, edge handling per step
    (4, 64, 256, 512, 264, (64, 1), (64, 1)),
    (3, 32, 300, 768, 520, (64, 4), (64, 3)),        # slices of three steps
    (2, 32, 130, 320, 2048, (64, 1), (64, 8)),
    (4, 32, 520, 2048, 2048, (64, 3), (64, 3)),      # two blocks per unit, eight rows in the last tile; uneven slices, added one by one
    (2, 64, 129, 4096, 1024, (64, 8), (64, 4)),      # one token in the last of three tiles
    (4, 32, 24, 1024, 64, (64, 4), (64, 1)),         # one K step
    (4, 40, 200, 640, 768, (64, 1), (64, 4)),        # group that no step is made of: general addressing
    (4, 32, 129, 512, 22016, (128, 1), (64, 16)),    # 128-row tiles, the second with one row
    (4, 32, 457, 256, 16496, (192, 1), (64, 16)),    # 192-row tiles that end past the padded copy
    (2, 32, 384, 256, 22016, (192, 1), (64, 16)),    # whole ones
]


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    lib = host_library(tmp_path_factory.mktemp("gemm_plan"), "gemm_plan", """
#include <algorithm>
#include "gemm_plan.hpp"
extern "C" int rows(int bits, int M, int N, int K, int g) { return qalora::gemm_dq_plan(bits, M, N, K, g).tile_rows; }
extern "C" int slices(int bits, int M, int N, int K, int g) { return qalora::gemm_dq_plan(bits, M, N, K, g).ksplit; }
extern "C" int general(int bits, int M, int N, int K, int g, int bwd) {
  const qalora::GemmPlan p = qalora::gemm_dq_plan(bits, M, N, K, g, bwd);
  return 100 * p.tile_rows + p.ksplit;
}
extern "C" size_t most(int bits, int M, int N, int K, int g, int bwd) { return qalora::gemm_dq_most_partials(bits, M, N, K, g, bwd); }
// of every batch of up to M tokens, one after the other
extern "C" size_t needed(int bits, int M, int N, int K, int g, int bwd) {
  size_t v = 0;
  for (int m = 1; m <= M; ++m) v = std::max(v, qalora::gemm_dq_partials(qalora::gemm_dq_plan(bits, m, N, K, g, bwd), m, N));
  return v;
}
extern "C" size_t room(int M, int N) { return qalora::gemm_dq_partial_room(M, N); }
extern "C" int fast(int K, int g) { return qalora::gemm_fast_shape(K, g); }
""")
    lib.room.restype = lib.most.restype = lib.needed.restype = ctypes.c_size_t
    return lib


def test_plans_are_launchable(plan):
    """A tile the kernel is built for, no empty slice, and partial sums within the room the workspace has."""
    rng = random.Random(3)
    for _ in range(3000):
        M, N = rng.choice([1, 16, 63, 64, 65, 128, 129, 192, 193, 4096, rng.randint(1, 9000)]), 8 * rng.randint(1, 2800)
        g = rng.choice([8, 24, 32, 64, 96, 128])
        K = 8 * rng.randint(1, 2800)
        bits = rng.choice([2, 3, 4])
        rows, ks = plan.rows(bits, M, N, K, g), plan.slices(bits, M, N, K, g)
        nk = -(-K // 64)
        assert rows in ((64, 128, 192, 256) if plan.fast(K, g) else (64, 128))
        assert 1 <= ks <= nk and -(-nk // -(-nk // ks)) == ks
        assert ks == 1 or 4 * ks * M * N <= plan.room(M, N)


@pytest.mark.parametrize("bits,group,tokens,d_in,d_out,fwd,bwd", SHAPES)
def test_plan_of(plan, bits, group, tokens, d_in, d_out, fwd, bwd):
    assert (plan.rows(bits, tokens, d_out, d_in, group), plan.slices(bits, tokens, d_out, d_in, group)) == fwd
    assert (plan.rows(bits, tokens, d_in, d_out, group), plan.slices(bits, tokens, d_in, d_out, group)) == bwd


@pytest.mark.parametrize("bits,tokens,d_in,d_out,group,bwd,best", [
    (4, 300, 4800, 11008, 96, 0, (64, 2)),      # us: 70, in (64, 1) 88
    (2, 512, 3072, 4096, 96, 0, (128, 4)),      # 37, in (64, 2) 41
    (3, 130, 13824, 2720, 32, 1, (128, 2)),     # 52, in (64, 3) 58
    (3, 100, 4096, 11000, 32, 1, (128, 16)),    # 43, in (64, 8) 45
])
def test_general_form_has_its_own_costs(plan, bits, tokens, d_in, d_out, group, bwd, best):
    N, K = (d_in, d_out) if bwd else (d_out, d_in)
    assert not plan.fast(K, group)
    assert divmod(plan.general(bits, tokens, N, K, group, bwd), 100) == best


def test_large_outputs_are_split(plan):
    # us: 421 in slices, 522 whole
    assert divmod(plan.general(3, 2048, 5120, 13800, 128, 1), 100)[1] > 1


def test_partials_of_shorter_batches(plan):
    """The room that a workspace has for partial sums is what some batch of up to its tokens needs."""
    rng = random.Random(9)
    for _ in range(150):
        M, N, K = rng.choice([1, 64, 65, 256, 300, 1000, rng.randint(1, 3000)]), 8 * rng.randint(1, 2800), 8 * rng.randint(1, 2800)
        args = (rng.choice([2, 3, 4]), M, N, K, rng.choice([32, 64, 96]), rng.randint(0, 1))
        assert plan.most(*args) == plan.needed(*args), args


@pytest.mark.parametrize("d_in,d_out", [(512, 512), (1024, 1024), (4096, 11008), (13824, 520), (22016, 8192), (1024, 8192)])
@pytest.mark.parametrize("bits,group", [(4, 32), (3, 64), (2, 128), (4, 8)])
def test_a_longer_batch_needs_no_less_workspace(d_in, d_out, bits, group):
    """One workspace sized for the longest batch serves the shorter ones.  (The backward with an adapter: test_grads_plan.)"""
    for op in (api.OP_FORWARD, api.OP_FORWARD_FACTORS16, api.OP_BACKWARD):
        sizes = [api.workspace_bytes(api.make_desc(d_in, d_out, bits, group), t, op) for t in (*range(1, 70), *range(70, 4200, 13))]
        assert sizes == sorted(sizes)


@pytest.mark.gpu
@pytest.mark.parametrize("bits,group,tokens,d_in,d_out,fwd,bwd", SHAPES)
def test_tiles_and_slices(gpu_api, bits, group, tokens, d_in, d_out, fwd, bwd):
    cfg = synth.LayerConfig("tiles", tokens, d_in, d_out, bits, group, 8, 0.5, seed=83)
    L = layer_on_gpu(gpu_api, cfg)
    d, n = L["desc"], L["np"]
    y = gpu_api.forward(d, L["x"], L["packed"], L["g_alpha"], L["g_beta"], L["A"], L["B"])
    ey = rel_err(y.cpu().numpy(), oracle.forward(n["x"], L["codes"], L["alpha"], L["beta"], group, n["A"], n["B"], cfg.s))
    dx, _, _ = gpu_api.backward(d, L["dy"], L["x"], L["packed"], L["g_alpha"], L["g_beta"], L["A"], L["B"])
    ref = oracle.backward(n["dy"], n["x"], L["codes"], L["alpha"], L["beta"], group, n["A"], n["B"], cfg.s)[0]
    ex = rel_err(dx.float().cpu().numpy(), ref)
    record(f"tiles {fwd} {bwd} b={bits} T={tokens} {d_in}x{d_out}", y=ey, dx=ex)
    assert ey <= 2e-3 and ex <= 2e-3
