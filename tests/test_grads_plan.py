"""Launch shapes of the adapters' gradients (host): the form that the sizes of the GPU tests take, and for sizes at
random that what the kernels are given fits: every unit in one run, no more partial sums of a tile than slots, runs of
dU's columns that end with them, and the room the workspace has."""
import random

import pytest

from host_code import host_library
from paper_2309_14717_amd import api
from test_gpu_grads import BY_U, SHAPES

FUSED, BY_Z, U = range(3)


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    return host_library(tmp_path_factory.mktemp("grads_plan"), "grads_plan", """
#include "grads_plan.hpp"
using namespace qalora;
extern "C" int form(int T, int L, int d_out, int rank) { return grads_plan(T, L, d_out, 1, &rank, &d_out).form; }
extern "C" int blocks(int T, int L, int d_out, int rank) { return grads_plan(T, L, d_out, 1, &rank, &d_out).runs.blocks; }
// 0, or what is wrong
extern "C" int check(int T, int L, int n, const int* rank, const int* part) {
  int d_out = 0;
  for (int q = 0; q < n; ++q) d_out += part[q];
  for (int f = 0; f < 3; ++f) {
    const GradsForm form = (GradsForm)f;
    const GradsPlan p = grads_plan(T, L, d_out, n, rank, part, &form);
    if (form == GRADS_FUSED) continue;
    const ZRuns& r = p.runs;
    if (r.blocks < 1 || r.first(0) != 0 || r.first(r.blocks) != r.units) return 1;
    for (int b = 0; b < r.blocks; ++b)
      if (r.first(b) >= r.first(b + 1) || r.owner(r.first(b)) != b || r.owner(r.first(b + 1) - 1) != b) return 2;
    for (int t = 0; t < r.units / r.steps; ++t)
      if (r.owner((t + 1) * r.steps - 1) - r.owner(t * r.steps) + 1 > p.slots) return 3;
    if (form != GRADS_BY_U) continue;
    for (int q = 0; q < n; ++q) {
      if (rank[q] > p.rank_tile) return 4;
      if (p.du_slices[q] < 1 || (p.du_slices[q] - 1) * p.du_steps * 64 >= part[q]) return 5;
      if (p.du_slices[q] * p.du_steps * 64 < part[q]) return 6;
      if ((size_t)p.du_slices[q] * T > grads_most_du_rows(T)) return 7;
      if (q && p.tile0[q] != p.tile0[q - 1] + ceil_div(part[q - 1], GZ_C)) return 8;
    }
    if (p.da_tokens % GA_T || p.da_shares > grads_most_da_shares(T, L, n)) return 9;
    if ((p.da_shares - 1) * p.da_tokens >= T || p.da_shares * p.da_tokens < T) return 10;
  }
  return 0;
}
""")


def test_forms(plan):
    for tokens, d_in, d_out, bits, group, rank in SHAPES:
        assert (plan.form(tokens, d_in // group, d_out, rank) == U) == ((tokens, rank) == (130, 8))
    for tokens, d_in, d_out, group, parts in BY_U:
        assert plan.form(tokens, d_in // group, d_out, max(r for _, r in parts)) == U
    # the benchmark's layers
    assert plan.form(64, 32, 1024, 16) == FUSED and plan.form(4096, 128, 4096, 64) == BY_Z
    assert plan.form(4096, 344, 4096, 64) == U and plan.form(4096, 8, 8192, 128) == BY_Z
    # measured: 7 to 20 % of the gradients' launches longer the other way
    assert plan.form(1531, 80, 13824, 64) == BY_Z and plan.form(700, 128, 4096, 16) == U
    assert plan.form(4096, 128, 22016, 64) == BY_Z and plan.form(4096, 128, 22016, 16) == U
    assert [plan.blocks(t, 128, 4096, 64) for t in (4096, 5952, 6016)] == [256, 256, 512]   # 2976 and 3008 units


def test_plans_are_launchable(plan):
    import ctypes
    rng = random.Random(7)
    for _ in range(4000):
        T = rng.choice([1, 63, 64, 65, 640, 641, 1024, 1025, rng.randint(1, 9000), rng.randint(1, 100000)])
        L, n = rng.randint(1, rng.choice([16, 140, 2000])), rng.choice([1, 1, 2, 3, 4])
        part = (ctypes.c_int * n)(*[8 * rng.randint(1, rng.choice([8, 300, 3000])) for _ in range(n)])
        rank = (ctypes.c_int * n)(*[rng.randint(1, 128) for _ in range(n)])
        assert plan.check(T, L, n, rank, part) == 0, (T, L, list(rank), list(part))


@pytest.mark.parametrize("d_in,d_out", [(512, 512), (4096, 4096), (4096, 11008), (11008, 4096), (13824, 2720), (4160, 40)])
@pytest.mark.parametrize("group,rank", [(8, 8), (32, 64), (32, 128)])
def test_a_longer_batch_needs_no_less_workspace(d_in, d_out, group, rank):
    tokens = list(range(1, 70)) + list(range(70, 1100, 17)) + [639, 640, 641, 1024, 1025, 2048, 4096, 5376, 5633, 8192, 65536, 70000]
    sizes = [api.workspace_bytes(api.make_desc(d_in, d_out, 4, group, rank, 0.5), t, api.OP_BACKWARD) for t in sorted(tokens)]
    assert sizes == sorted(sizes)
