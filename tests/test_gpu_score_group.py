"""The 16-bit scoring kernels at the edges of their splits: more than 128 window rows per KV head (tiles in sets of four
that all wavefronts share) in both orders of pooling and averaging, and the row-pooling order for fewer rows (tiles
that overlap by the pool radius): sequences shorter than a tile or a set, one key more, odd rows, every radius that is
pooled in registers, and row weights that differ from key to key so that a misplaced maximum shows."""
import numpy as np
import pytest
import torch

import paper_2407_11550_amd as adakv
from paper_2407_11550_amd import synth

DEV = "cuda:0"

# h_q, h_kv, d, w, n, dtype; pool kernels
CASES = [
    (4, 2, 128, 66, [1, 31, 33, 127, 128, 129, 400], torch.bfloat16, (1, 7)),    # 132 rows
    (10, 2, 128, 51, [1000, 5], torch.float16, (5,)),                            # 255 rows: the last pair of partials is half a pair
    (4, 2, 64, 100, [513, 97], torch.bfloat16, (13,)),                           # 200 rows
    (16, 2, 128, 64, [700, 3, 161], torch.bfloat16, (7, 15)),                    # 512 rows
    (10, 2, 64, 60, [900, 32], torch.float16, (7,)),                             # 300 rows, d = 64
    (128, 64, 128, 100, [1500], torch.bfloat16, (7,)),                           # 200 rows, several sets per workgroup
    (128, 64, 64, 129, [1100, 64], torch.bfloat16, (3,)),                        # 258 rows, d = 64
    (2, 2, 128, 1, [1, 2, 26, 27, 53, 100], torch.bfloat16, (7, 15)),            # one row; a tile's own 26 keys, and one more
    (8, 2, 64, 32, [500, 18, 33], torch.float16, (1, 3, 9, 11)),                 # 128 rows
    (256, 64, 128, 32, [1300, 7], torch.bfloat16, (5, 13)),
]


def _reference(wl, q, K, pool_first, lse=None):
    out, bound, scale = [], 0.0, 1.0 / np.sqrt(wl.d)
    pool = torch.nn.functional.max_pool1d
    for b, n in enumerate(wl.n):
        qb, Kb = q[b].double(), K[wl.tok_off[b]:wl.tok_off[b] + n].double()
        for c in range(wl.h_kv):
            rows, keys = qb[c * wl.g:(c + 1) * wl.g].reshape(-1, wl.d), Kb[:, c].t().contiguous()
            bound = max(bound, float((scale * rows.abs() @ keys.abs()).max()))
            logits = scale * rows @ keys
            a = torch.softmax(logits, dim=1) if lse is None else torch.exp(logits - lse[b, c * wl.g:(c + 1) * wl.g].reshape(-1, 1).double())
            if pool_first:
                out.append(pool(a[None], wl.pool_k, 1, wl.pool_k // 2)[0].mean(0))
            else:
                out.append(pool(a.mean(0)[None, None], wl.pool_k, 1, wl.pool_k // 2)[0, 0])
    # a logit is a sum of d products rounded d times, then scaled: off by at most (d + 4) 2^-24 times the sum of the
    # products' magnitudes, the log-sum-exp by no more; 1e-6 covers the exponential, the logarithm and the sums over rows
    return torch.cat(out).cpu().numpy(), 2 * (wl.d + 4) * 2.0 ** -24 * bound + 1e-6


@pytest.mark.gpu
@pytest.mark.parametrize("given_lse", [False, True], ids=["sweep", "row_lse"])
@pytest.mark.parametrize("pool_first", [False, True], ids=["mean_first", "pool_first"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "hq%d_h%d_d%d_w%d_n%s" % (c[:4] + ("-".join(map(str, c[4][:4])),)))
def test_scores_at_the_edges(case, pool_first, given_lse):
    h_q, h, d, w, n, dt, pools = case
    for k in pools:
        print("sets and overlapping tiles", case[:5], k, pool_first, given_lse, flush=True)
        wl = synth.small_workload(h_q, h, d, w, k, n, [h * w] * len(n), dtype=dt, seed=43, temps=(0.25, 1.0))
        q, K, _ = synth.generate(wl, device=DEV)
        layer = adakv.Layer.from_workload(wl, flags=4 if pool_first else 0)
        assert adakv.describe(layer)["score"] == ("mfma-pool-first" if pool_first else "mfma")
        out = torch.full((layer.num_scores + 64,), -7.0, device=DEV)      # canaries behind the scores
        ws = torch.full((adakv.workspace_bytes(layer),), 0xFF, dtype=torch.uint8, device=DEV)
        lse = synth.prefill_row_lse(wl, q, K) if given_lse else None
        adakv.score(layer, q, K, row_lse=lse, out=out, ws=ws)
        got = out.cpu().numpy().astype(np.float64)
        want, tol = _reference(wl, q, K, pool_first, lse)
        assert tol < 2e-3 and np.all(got[layer.num_scores:] == -7.0)
        err = np.abs(got[:layer.num_scores] - want) / want
        assert err.max() <= tol, (k, err.max(), tol)


@pytest.mark.gpu
@pytest.mark.parametrize("h_q,d,w,dt", [(2, 64, 20, torch.float16), (8, 128, 32, torch.bfloat16), (16, 128, 31, torch.bfloat16),
                                        (16, 64, 64, torch.bfloat16)], ids=["20rows", "128rows", "248rows", "512rows"])
def test_a_nan_key_spoils_every_window_that_holds_it(h_q, d, w, dt):
    """The row-pooling order with a log-sum-exp from elsewhere: a key that is a NaN, of either sign, makes the scores
    within the pool radius of it in its head -inf, so that none of them is kept, and no other."""
    h, n, k = 2, 700, 7
    print("a NaN in the row-pooling order", h_q, d, w, flush=True)
    wl = synth.small_workload(h_q, h, d, w, k, [n], [h * w], dtype=dt, seed=47)
    q, K, _ = synth.generate(wl, device=DEV)
    lse = synth.prefill_row_lse(wl, q, K)
    layer = adakv.Layer.from_workload(wl, flags=4)
    assert adakv.describe(layer)["score"] == "mfma-pool-first"
    clean = adakv.score(layer, q, K, row_lse=lse).reshape(h, n)
    assert bool(torch.isfinite(clean).all())
    for at, sign in ((0, 1), (15, -1), (16, 1), (28, 1), (31, -1), (32, 1), (333, -1), (n - 1, 1)):
        bad = K.clone()
        bits = 0x7E00 if dt == torch.float16 else 0x7FC0
        bad.view(torch.int16)[at, 1, d // 3] = bits if sign > 0 else bits - 0x8000
        got = adakv.score(layer, q, bad, row_lse=lse).reshape(h, n)
        want = torch.zeros((h, n), dtype=torch.bool, device=DEV)
        want[1, max(at - k // 2, 0):at + k // 2 + 1] = True
        assert torch.equal(got == -torch.inf, want), (at, (got == -torch.inf).nonzero().tolist())
        assert torch.equal(got[~want], clean[~want]), at
