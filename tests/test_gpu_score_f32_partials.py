"""The fp32 scoring kernels between 4097 and 8192 keys: statistics per 256 keys, at most 32 of them, which the weights
sweep combines itself where that leaves no compute unit with much more to do."""
import pytest
import torch

import paper_2407_11550_amd as adakv
from paper_2407_11550_amd import synth
from test_gpu_score_f32 import test_fp32_scoring_at_the_edges_of_its_split as _score_and_compare

# h_q, h_kv, d, w, n per sequence, who combines the partials
CASES = [
    (4, 2, 64, 8, [4097], "fused"),                 # 17 partials, the last of one key
    (4, 2, 64, 8, [8192, 5, 4097, 256], "fused"),   # 32, and sequences with one
    (4, 2, 64, 8, [8193], "kernel"),
    (4, 2, 128, 32, [6000], "kernel"),              # two row blocks, d = 128: half as many workgroups would take too long
    (16, 8, 128, 32, [5000], "fused"),              # two workgroups of four wavefronts, or one of eight, on the fullest
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "h%d_d%d_w%d_n%s" % (c[1:4] + ("-".join(map(str, c[4])),)))
def test_who_combines(case):
    h_q, h, d, w, n, who = case
    wl = synth.small_workload(h_q, h, d, w, 7, n, [h * w] * len(n), dtype=torch.float32)
    assert adakv.describe(adakv.Layer.from_workload(wl))["lse"] == who


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda c: "h%d_d%d_w%d_n%s" % (c[1:4] + ("-".join(map(str, c[4])),)))
def test_scores(case):
    h_q, h, d, w, n, _ = case
    _score_and_compare((h_q, h, d, w, 7, n, torch.float32, "fused"), False)
