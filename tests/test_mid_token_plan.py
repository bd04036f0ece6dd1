"""The launch shape of the mid-token forward: the search that ends early finds what pricing every block count
finds, in less host time (every call makes it)."""
import ctypes
import random

import pytest

from host_code import host_library
from paper_2309_14717_amd import api

HEAD, PARTIAL = 2304, 4 * 8192   # flags and status word; the partial of a block at 64 tokens


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    lib = host_library(tmp_path_factory.mktemp("plan"), "plan", """
#include <chrono>
#include "midt_plan.hpp"
using namespace qalora;
extern "C" int blocks(int bits, int d_in, int d_out, int tokens, size_t scratch) {
  return midt_blocks(bits, d_in, d_out, tokens, scratch);
}
// every count from one up, the smallest of equally cheap ones
extern "C" int full_search(int bits, int d_in, int d_out, int tokens, size_t scratch) {
  const int CU = ceil_div(d_in / 128, MT_DEEP), S = ceil_div(d_out, MT_SLAB);
  const int units = S * CU;
  const int tt = midt_tiles(tokens);
  const long room = scratch <= ST_HEAD_BYTES ? 0 : (long)((scratch - ST_HEAD_BYTES) / ((size_t)tt * 4 * 128 * 16));
  int best = 0;
  double best_cost = 0, free_cost = 0;
  for (int nb = 1; nb <= ST_MAX_BLOCKS && nb <= units; ++nb) {
    const bool whole = midt_whole_slabs(CU, S, nb);
    const double cost = midt_cost(units, CU, S, midt_unit(bits, tt), tt, nb, ceil_div(nb, S));
    if (free_cost == 0 || cost < free_cost) free_cost = cost;
    if ((whole || nb <= room) && (best == 0 || cost < best_cost)) {
      best = nb;
      best_cost = cost;
    }
  }
  return best > 0 && best_cost <= midt_short_of(bits) * free_cost ? best : 0;
}
extern "C" double us_per_call(int full, int d_in, int d_out) {
  volatile int sink = 0;
  const auto t0 = std::chrono::steady_clock::now();
  for (int i = 0; i < 1000; ++i) sink = sink + (full ? full_search : blocks)(4, d_in, d_out, 64, 1ul << 30);
  return std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count() / 1000;
}
""")
    lib.us_per_call.restype = ctypes.c_double
    return lib


def test_early_end_changes_no_plan(plan):
    rng = random.Random(5)
    shapes = [(4096, 4096), (8192, 22016), (22016, 8192), (5120, 13824), (128, 8), (128, 22016), (1024, 520), (65536, 8192)]
    shapes += [(128 * rng.randint(1, 172), 8 * rng.randint(1, 2752)) for _ in range(400)]
    shapes += [(128 * rng.randint(1, 40), 8 * rng.randint(1, 600)) for _ in range(400)]
    for d_in, d_out in shapes:
        for tokens in (5, 33, 64):
            for scratch in (0, HEAD, HEAD + 256 * PARTIAL, rng.randint(HEAD, HEAD + 256 * PARTIAL),
                            (d_in // rng.choice([32, 64, 128]) + 1) * d_out * 4):
                args = (rng.choice([2, 3, 4]), d_in, d_out, tokens, ctypes.c_size_t(scratch))
                assert plan.blocks(*args) == plan.full_search(*args), args[:4] + (scratch,)


@pytest.mark.parametrize("bits,d_in,d_out,tokens,blocks", [
    (4, 2048, 8192, 64, 192), (4, 8192, 8192, 64, 256), (2, 8192, 8192, 24, 256), (3, 8192, 8192, 53, 256),
])
def test_counts_that_measured_best(plan, bits, d_in, d_out, tokens, blocks):
    """A multiple of the slabs' number cuts every slab into as many parts and no run crosses one, whether or
    not the parts are equally long (2048 x 8192: three parts of four units).  While only equal parts were
    taken to stay inside a slab 248 blocks were chosen at the first two: 18.9 and 32.2 us against 18.2
    and 29.6."""
    assert plan.blocks(bits, d_in, d_out, tokens, ctypes.c_size_t(HEAD + 256 * PARTIAL)) == blocks


@pytest.mark.parametrize("d_in,d_out", [(8192, 8192), (8192, 22016), (65536, 8192)])
def test_search_is_shorter(plan, d_in, d_out):
    full, early = (min(plan.us_per_call(f, d_in, d_out) for _ in range(7)) for f in (1, 0))
    print(f"plan {d_in}x{d_out}: {early:.2f} us, all counts {full:.2f}")
    assert early < 0.75 * full


@pytest.mark.parametrize("group", [32, 64, 128])
def test_the_workspace_leaves_room_for_any_count(plan, group):
    """The dense kernel's room for slices alone, in proportion to the tokens, was too little for few of them: 4096 x 4096
    deployed at 5 tokens ran on 128 blocks where 224 are the cheapest, and with groups of 128 on the dense kernel."""
    for bits in (4, 3, 2):
        for d_in in range(1024, 8193, 512):
            for d_out in (8, 512, 1032, 2048, 2720, 4096, 8192):
                desc = api.make_desc(d_in, d_out, bits, group)
                for tokens in (5, 6, 8, 11, 16, 17, 32, 33, 48, 49, 64):
                    free = plan.blocks(bits, d_in, d_out, tokens, ctypes.c_size_t(1 << 30))
                    assert api.mid_blocks(desc, tokens) == free > 0
