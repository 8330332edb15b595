"""Top-k scopes spread over the chip: the gather kernel's 1024 threads, and emit with 1024, 512 and 256 of them by the
number of blocks, against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import paper_2407_11550_amd as adakv
from oracle import adakv_oracle as O

from test_gpu_topk_block import DEV, _scores

pytestmark = pytest.mark.gpu

# KV heads, prefix lengths: blocks of 4096 positions
LAYERS = [
    (1, [16385]),                     # 5
    (8, [20480, 20481, 1]),           # whole chunks, a chunk of one position, a sequence of one
    (32, [32768]),                    # 256: the last with 1024 threads
    (33, [32767]),                    # 264: 512 threads
    (64, [32768]),                    # 512: the last with 512
    (64, [16400, 16385]),             # 640: 256 threads, two sequences
]


@pytest.mark.parametrize("kind", ["spread", "pooled", "equal", "one_prefix", "signed"])
@pytest.mark.parametrize("h,lengths", LAYERS, ids=lambda v: str(v))
def test_budgets_and_positions(h, lengths, kind):
    print("topk spread", h, lengths, kind, flush=True)
    rng = np.random.default_rng(h + len(kind))
    w, alpha = 2, 0.2
    sc = [rng.standard_normal((h, n)).astype(np.float32) if kind == "signed" else _scores(rng, kind, h, n) for n in lengths]
    for keep in (0.001, 0.3):
        B = [h * w + int(keep * h * n) for n in lengths]
        layer = adakv.Layer(torch.bfloat16, h, h, 64, w, 7, alpha, lengths, B)
        flat = torch.from_numpy(np.concatenate([s.reshape(-1) for s in sc])).to(DEV)
        bud, cu = adakv.allocate(layer, flat)
        guard = torch.full((sum(B) + 256,), -5, dtype=torch.int32, device=DEV)
        adakv.select(layer, flat, bud, cu, indices=guard)
        got, row = guard.cpu().numpy(), 0
        assert np.all(got[sum(B):] == -5)
        for b, n in enumerate(lengths):
            want, _ = O.allocate(sc[b], B[b], w, alpha)
            assert np.array_equal(bud.cpu().numpy()[b * h:(b + 1) * h], want)
            assert np.array_equal(got[row:row + B[b]], O.select(sc[b], want, w))
            row += B[b]
