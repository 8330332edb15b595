"""The kernel that works out a sequence's budgets and gathers for a head in one launch: where it is taken, and that
the step gives there what the two self-contained calls give on the same scores."""
import pytest
import torch

import paper_2407_11550_amd as adakv
from paper_2407_11550_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ONE, TWO = ["alloc_gather", "topk_finish_gather", "select_emit"], ["alloc_gather", "alloc_finish", "select_gather", "select_emit"]

# query heads, KV heads, window, prefix lengths, share kept, all keys zero (every score the same), kernels
CASES = [
    (4, 4, 4, [12288], 0.05, False, ONE),                 # whole chunks of 4096
    (4, 4, 4, [12289], 0.3, False, ONE),                  # a chunk of one position
    (16, 4, 32, [30000, 300, 4097, 1], 0.0, False, ONE),    # no budget beside the window: nothing to gather
    (16, 4, 32, [28673, 300, 4097, 1], 0.1, False, ONE),  # sequences of one chunk beside a long one
    (4, 4, 4, [10000], 1.0, False, ONE),                  # everything is kept
    (4, 4, 4, [20000], 0.1, True, ONE),                   # a plateau
    (64, 64, 1, [10000], 0.02, False, ONE),               # 192 blocks of 64 heads
    (8, 8, 2, [131072], 0.01, False, ONE),                # 256 blocks
    (8, 8, 2, [131073], 0.01, False, TWO),                # 264
    (3, 3, 4, [20000], 0.05, False, TWO),                 # three segments
    (4, 4, 1, [8193], 0.05, False, TWO),                  # the lists do not fit beside so few scores ...
    (32, 4, 16, [8193], 0.05, False, ONE),                # ... until the partial statistics of 128 rows make room
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "h%d_w%d_n%s_keep%s%s" % (c[1], c[2], "-".join(map(str, c[3])), c[4], "_flat" * c[5]))
def test_the_step_gives_what_the_two_calls_give(case):
    h_q, h, w, n, keep, flat, kernels = case
    print("finish and gather", case, flush=True)
    wl = synth.small_workload(h_q, h, 64, w, 7, n, [h * w + int(keep * h * nb) for nb in n], seed=23)
    q, K, V = synth.generate(wl, device=DEV)
    if flat:
        K.zero_()
    layer = adakv.Layer.from_workload(wl)
    ws = torch.full((adakv.workspace_bytes(layer),), 0xAB, dtype=torch.uint8, device=DEV)
    with adakv.KernelTrace(64) as tr:
        out = adakv.compress(layer, q, K, V, ws=ws)
    torch.cuda.synchronize()
    assert [k for k, _ in tr.durations_us() if k.split("_")[0] in ("topk", "alloc", "select")] == kernels
    bud, cu = adakv.allocate(layer, out["scores"])
    idx = adakv.select(layer, out["scores"], bud, cu)
    assert torch.equal(out["budgets"], bud) and torch.equal(out["cu_seqlens"], cu) and torch.equal(out["indices"], idx)
