"""The 16-bit scoring kernels for up to 128 window rows per KV head, whose wavefronts take tiles of 32 keys on
their own: which tiles and rows they ask for (a model on the CPU), and scores at the edges of the split: fewer
tiles than wavefronts, a last tile of one key, odd rows (the statistics are combined in pairs), sequences long
enough that the first tile's maxima serve as the reference of all, and logits that overflow it."""
import numpy as np
import pytest
import torch

import paper_2407_11550_amd as adakv
from paper_2407_11550_amd import synth

from test_gpu_score_f32 import _reference

DEV = "cuda:0"
TILE, NW = 32, 4


def rows_asked(key0, lo, hi):
    """The rows a tile's lanes ask for: 32 from key0 on, clamped to [lo, hi] (all of them as they are inside)."""
    key0 = min(key0, hi)
    return [key0 + max(min(r, hi - key0), max(lo - key0, 0)) for r in range(TILE)]


@pytest.mark.parametrize("nch", [1, 2, 7, 32])
def test_statistics_tiles_are_dealt_out_once(nch):
    for n in [1, 31, 32, 33, 127, 128, 129, 1000, 4096, 4097]:
        ntiles, taken = -(-n // TILE), []
        for chunk in range(nch):
            for wv in range(NW):
                first, stride = chunk * NW + wv, nch * NW
                iters = (ntiles - 1 - first) // stride + 1 if first < ntiles else 0
                mine = [first + it * stride for it in range(iters)]
                taken += mine
                for t in mine[:-1]:
                    assert (t + 1) * TILE <= n                     # only a wavefront's last tile can be ragged
                for t in mine:
                    assert all(0 <= r < n for r in rows_asked(t * TILE, 0, n - 1))
        assert sorted(taken) == list(range(ntiles))


@pytest.mark.parametrize("pool_r,fused", [(0, True), (3, True), (32, True), (0, False)])
@pytest.mark.parametrize("chunk_len", [64, 96, 128, 448, 3840])
def test_weights_tiles_cover_a_chunk_and_its_halo(chunk_len, pool_r, fused):
    for n in [1, 33, 63, 64, 65, 129, 3839, 3841, 5000]:
        nch = -(-n // chunk_len)
        for chunk in range(nch):
            kc0, kc1 = chunk * chunk_len, min(n, (chunk + 1) * chunk_len)
            k0 = kc0 - TILE if fused and kc0 > 0 else kc0
            k1 = min(n, kc1 + pool_r) if fused else kc1
            lo, hi = max(kc0 - pool_r, 0), min(kc1 - 1 + pool_r, n - 1)
            ntiles, taken = -(-(k1 - k0) // TILE), []
            assert ntiles * TILE <= chunk_len + 2 * TILE           # the scores' place in LDS
            for wv in range(NW):
                iters = (ntiles - 1 - wv) // NW + 1 if wv < ntiles else 0
                rot = chunk * iters // nch
                for it in range(iters):
                    p = rot - 1 - it
                    taken.append(wv + (p + iters if p < 0 else p) * NW)
                asked = rows_asked(k0 + taken[-1] * TILE if iters else k0, lo, hi)      # (asked for without tiles too)
                assert all(0 <= r < n for r in asked)
            assert sorted(taken) == list(range(ntiles))
            for t in taken:
                asked = rows_asked(k0 + t * TILE, lo, hi)
                assert all(0 <= r < n for r in asked)
                for j, r in enumerate(asked):                       # every key somebody needs is itself
                    if lo <= k0 + t * TILE + j <= hi:
                        assert r == k0 + t * TILE + j


# h_q, h_kv, d, w, pool_k, n, dtype
CASES = [
    (2, 2, 128, 1, 1, [1, 2, 31, 32, 33, 64, 65], torch.bfloat16),      # one row, a few keys
    (3, 1, 64, 1, 7, [3000], torch.float16),                            # three rows
    (2, 2, 128, 127, 7, [700, 5], torch.bfloat16),                      # 127 rows: the last pair is half a pair
    (4, 2, 64, 17, 65, [2000, 97], torch.bfloat16),                     # 34 rows, the largest pool that is fused
    (4, 2, 128, 48, 71, [900], torch.float16),                          # 96 rows, the pool in its own kernel
    (64, 64, 128, 32, 7, [2049], torch.bfloat16),                       # kept reference, last tile of one key
    (128, 64, 64, 25, 5, [2600, 33], torch.float16),
    (256, 64, 128, 32, 7, [2080, 1, 2049], torch.bfloat16),
    (256, 64, 64, 32, 13, [4127], torch.bfloat16),
]


@pytest.mark.gpu
@pytest.mark.parametrize("given_lse", [False, True], ids=["sweep", "row_lse"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "hq%d_h%d_d%d_w%d_k%d_n%s_%s" % (c[:5] + ("-".join(map(str, c[5])), str(c[6])[6:])))
def test_scores_at_the_edges_of_the_split(case, given_lse):
    h_q, h, d, w, k, n, dt = case
    print("own tiles", case, given_lse, flush=True)
    wl = synth.small_workload(h_q, h, d, w, k, n, [h * w] * len(n), dtype=dt, seed=37, temps=(0.25, 1.0))
    q, K, _ = synth.generate(wl, device=DEV)
    lse = synth.prefill_row_lse(wl, q, K) if given_lse else None
    layer = adakv.Layer.from_workload(wl)
    assert adakv.describe(layer)["score"] == "mfma"
    out = torch.full((layer.num_scores + 64,), -7.0, device=DEV)          # canaries behind the scores
    ws = torch.full((adakv.workspace_bytes(layer),), 0xFF, dtype=torch.uint8, device=DEV)
    adakv.score(layer, q, K, row_lse=lse, out=out, ws=ws)
    got = out.cpu().numpy().astype(np.float64)
    want, tol = _reference(wl, q, K, lse)     # its bound holds for any order of fp32 sums of d exact or rounded products
    assert tol < 2e-3 and np.all(got[layer.num_scores:] == -7.0)
    err = np.abs(got[:layer.num_scores] - want) / want
    assert err.max() <= tol, (err.max(), tol)


@pytest.mark.gpu
@pytest.mark.parametrize("h_q,w", [(64, 8), (256, 32)])                   # 8 rows, 128 rows
def test_logits_far_above_the_kept_reference(h_q, w):
    """Every wavefront's first tile has tiny keys, later ones logits more than 128 powers of two above them: the sums
    overflow and are taken again with a running maximum."""
    print("own tiles, overflow", h_q, w, flush=True)
    h, n, d = 64, 2500, 128
    wl = synth.small_workload(h_q, h, d, w, 7, n, h * w, dtype=torch.bfloat16, seed=41)
    q, K, _ = synth.generate(wl, device=DEV)
    q = (q.float() * 4).to(torch.bfloat16)
    K = K.float()
    K[:1024] *= 0.01
    K[1024:] *= 6
    K = K.to(torch.bfloat16)
    rows = q[0, :h_q // h].reshape(-1, d).float()
    logits = rows @ K[:n, 0].float().t().contiguous() / d ** 0.5
    assert float((logits[:, 1024:].amax(1) - logits[:, :1024].amax(1)).max()) * 1.4427 > 128
    got = adakv.score(adakv.Layer.from_workload(wl), q, K).cpu().numpy().astype(np.float64)
    want, tol = _reference(wl, q, K)
    big = want > 1e-30                                                    # (weights below 2^-126 are zero in these kernels)
    assert np.all(np.isfinite(got)) and np.all(np.abs(got - want)[big] <= tol * want[big])
    assert np.all(got[~big] <= 1e-30 * (1 + tol))
