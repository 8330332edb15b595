"""Pooling in every window row before the mean: the radii on both sides of the line between steps of one key and of
two (3), odd and even ones, in every layout of the matrix-core sweep, with lengths that end inside a tile."""
import pytest
import torch

import paper_2407_11550_amd as adakv
from paper_2407_11550_amd import synth
from paper_2407_11550_amd.binding import ADAKV_FLAG_POOL_THEN_MEAN
from oracle import adakv_oracle as O
from parity_util import assert_scores_close, to_f64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("radius", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("h_q,h,d,w,n", [
    (2, 2, 128, 32, [1, 300]),                 # 32 rows
    (4, 2, 64, 25, [19, 333]),                 # 50
    (8, 2, 128, 32, [33, 1111]),               # 128
    (8, 2, 64, 31, [18, 700]),                 # 124
    (16, 2, 128, 32, [17, 901]),               # 256
    (16, 1, 128, 31, [32, 401]),               # 496
    (16, 1, 64, 32, [31, 403]),                # 512
])
def test_radii(h_q, h, d, w, n, radius):
    print("pool rows", h_q, h, d, w, n, radius, flush=True)
    k = 2 * radius + 1
    wl = synth.small_workload(h_q, h, d, w, k, n, [h * w] * len(n), dtype=torch.bfloat16, seed=radius)
    q, K, _ = synth.generate(wl, device=DEV)
    got = adakv.score(adakv.Layer.from_workload(wl, flags=ADAKV_FLAG_POOL_THEN_MEAN), q, K).cpu().numpy()
    at = 0
    for b in range(wl.batch):
        keys = to_f64(K[wl.tok_off[b]:wl.tok_off[b + 1]])
        want = O.score(to_f64(q[b]), keys, wl.n[b], w, k, order="pool_then_mean")
        assert_scores_close(got[at:at + h * wl.n[b]], want, f"seq {b}")
        at += h * wl.n[b]
