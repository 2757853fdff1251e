"""GPU parity at the sizes where a launch changes its shape: edges of tiles, remainders, the lines of the
dispatch rules.  Same oracle, same tolerances as test_gpu_parity.py."""

import numpy as np
import pytest

from oracle import ppmoe_oracle as O
from paper_2304_11414_amd import synth
from tests.test_gpu_parity import check_dispatch, compare_layer_full, small_cfg

pytestmark = pytest.mark.gpu


# ---------------------------------------------------------------- permutation and balance loss

@pytest.mark.parametrize("kw", [
    dict(T=64 * 4096, E=8, top_k=1),                                # 4096 segments: the last the placing kernel scans
    dict(T=64 * 4096 + 1, E=8, top_k=1, capacity_factor=1.0),       # one more: the scan is a launch of its own
    dict(T=64 * 15 + 1, E=17, top_k=1),                             # 16 segments = one block; two rounds of experts
    dict(T=32769, E=130, top_k=2, local_begin=1, local_count=129),
])
def test_dispatch_at_the_lines_of_the_scan(kw):
    lc = small_cfg(d=64, **kw)
    idx = O.top_k_picks(synth.random_logits(lc.T, lc.E, seed=lc.T), lc.top_k)
    check_dispatch(lc, idx)


@pytest.mark.parametrize("kw", [
    dict(T=3000, d=128, F=128, E=12, top_k=2, renorm_topk=True, seed=61),    # slices of 12 threads, some idle
    dict(T=700, d=128, F=128, E=100, top_k=2, local_begin=20, local_count=10, seed=62),
    dict(T=130, d=128, F=128, E=256, top_k=1, local_begin=0, local_count=16, seed=63),
])
def test_balance_loss_inside_the_layer(kw):
    lc = small_cfg(**kw)
    compare_layer_full(lc, synth.make_inputs(lc))
