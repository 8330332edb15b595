"""The scoring kernels that multiply and accumulate in fp32 (fp32 inputs, and 16-bit inputs beyond
512 window rows per KV head) at the edges of their split: 128 keys per workgroup of which
128 - 2*radius are owned when the pool is applied in the sweep, 32 keys per wavefront, window rows
32 at a time, the pool in a kernel of its own beyond radius 16, statistics per 256 keys where the
scratch memory for a 128-key split would pass the built-in array."""
import numpy as np
import pytest
import torch

import paper_2407_11550_amd as adakv
from oracle import adakv_oracle as O
from paper_2407_11550_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# h_q, h_kv, d, w, pool_k, n per sequence, dtype, where the pool runs
CASES = [
    (4, 4, 64, 8, 7, [1, 31, 32, 33], torch.float32, "fused"),            # fewer keys than a wavefront holds; one row block
    (4, 2, 128, 16, 7, [121, 122, 123, 128, 129], torch.float32, "fused"),  # around the owned 122 and the held 128 keys
    (4, 4, 128, 1, 1, [127, 257], torch.float32, "fused"),                # one row, no pool: all 128 keys owned
    (4, 2, 64, 20, 7, [4096, 5, 3000], torch.float32, "fused"),           # 32 partials per row: combined in sweep 2
    (4, 2, 64, 20, 7, [5, 4097], torch.float32, "fused"),                 # 33: by a kernel
    (12, 4, 64, 11, 5, [500, 77], torch.float32, "fused"),                # 33 rows: a row block with one row
    (2, 1, 128, 32, 33, [97, 300], torch.float32, "fused"),               # radius 16: 96 owned keys
    (2, 1, 128, 32, 35, [300], torch.float32, "kernel"),                   # radius 17: the pool in its own kernel
    (16, 2, 128, 64, 7, [1300], torch.float32, "fused"),                  # 512 rows
    (18, 2, 64, 64, 13, [250, 1000], torch.bfloat16, "fused"),            # 576 rows of 16-bit inputs
    (18, 2, 128, 64, 7, [245], torch.float16, "fused"),
    (64, 64, 128, 96, 7, [500], torch.float32, "kernel"),                  # 320 workgroups with the pool, 256 without: its own kernel
    (32, 32, 64, 2, 7, [251 + b % 11 for b in range(64)], torch.float32, "fused"),   # 2048 heads: 256-key statistics
    (32, 32, 128, 2, 7, [251 + b % 11 for b in range(64)], torch.float32, "kernel"),
]


def _reference(wl, q, K, lse=None):
    off, out, bound = wl.tok_off, [], 0.0
    scale = 1.0 / np.sqrt(wl.d)
    for b, n in enumerate(wl.n):
        qb, Kb = q[b].double().cpu().numpy(), K[off[b]:off[b] + n].double().cpu().numpy()
        for c in range(wl.h_kv):
            rows = qb[c * wl.g:(c + 1) * wl.g].reshape(-1, wl.d)
            s = scale * rows @ Kb[:, c].T
            bound = max(bound, float((scale * np.abs(rows) @ np.abs(Kb[:, c]).T).max()))
            m = s.max(axis=1, keepdims=True)
            z = np.log(np.exp(s - m).sum(axis=1, keepdims=True)) + m if lse is None else \
                lse[b, c * wl.g:(c + 1) * wl.g].double().cpu().numpy().reshape(-1, 1)
            out.append(O.max_pool_same(np.exp(s - z).mean(axis=0)[None], wl.pool_k)[0])
    # A logit is a sum of d products rounded d times, then scaled: off by at most (d + 4) 2^-24 times
    # the sum of the products' magnitudes; the log-sum-exp is off by no more, and the exponential
    # passes both on relatively.  1e-6 covers the exponential, the logarithm and the sums over rows.
    return np.concatenate(out), 2 * (wl.d + 4) * 2.0 ** -24 * bound + 1e-6


@pytest.mark.parametrize("given_lse", [False, True], ids=["sweep", "row_lse"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "hq%d_h%d_d%d_w%d_k%d_n%s_%s" % (c[:5] + ("-".join(map(str, c[5][:5])), str(c[6])[6:])))
def test_fp32_scoring_at_the_edges_of_its_split(case, given_lse):
    h_q, h, d, w, k, n, dt, pool = case
    print("fp32 scoring", case, given_lse, flush=True)
    wl = synth.small_workload(h_q, h, d, w, k, n, [h * w] * len(n), dtype=dt, seed=31, temps=(0.25, 1.0))
    q, K, _ = synth.generate(wl, device=DEV)
    lse = synth.prefill_row_lse(wl, q, K) if given_lse else None
    layer = adakv.Layer.from_workload(wl)
    desc = adakv.describe(layer)
    assert desc["score"] == "fma" and desc["pool"] == pool
    out = torch.full((layer.num_scores + 64,), -7.0, device=DEV)          # canaries behind the scores
    adakv.score(layer, q, K, row_lse=lse, out=out)
    got = out.cpu().numpy().astype(np.float64)
    want, tol = _reference(wl, q, K, lse)
    assert tol < 2e-3 and np.all(got[layer.num_scores:] == -7.0)
    err = np.abs(got[:layer.num_scores] - want) / want
    assert err.max() <= tol, (err.max(), tol)


@pytest.mark.parametrize("given_lse", [False, True], ids=["sweep", "row_lse"])
@pytest.mark.parametrize("w,n", [(16, 300), (5, 300), (16, 5000)])       # 32 rows; 10; statistics combined by a kernel
def test_weights_below_the_normal_range_keep_their_order(w, n, given_lse):
    """One key takes all of the softmax, the others' weights are exp(-87.5) to exp(-102.5), 2^-126 to 2^-148:
    scores of subnormal weights, not ties at zero.  A weight's exponent of up to 148 is rounded to 2^-24 of
    itself in the logit, the scaling and the log-sum-exp, 148 ln 2 * 3 * 2^-24 = 1.8e-5 of the weight, and
    a subnormal sum, mean and conversion to half a unit of 2^-149 each."""
    print("fp32 small weights", w, n, given_lse, flush=True)
    h, g, d = 2, 2, 64
    rng = np.random.default_rng(n + w)
    K = torch.zeros((n + w, h, d), device=DEV)
    K[:, :, 0] = torch.from_numpy(-(87.5 + 15 * rng.random((n + w, h))).astype(np.float32)).to(DEV)
    K[n // 2, :, 0] = 0.0
    q = torch.zeros((1, g * h, w, d), device=DEV)
    q[..., 0] = 1.0
    layer = adakv.Layer(torch.float32, g * h, h, d, w, 1, 0.2, [n], [h * w], scale=1.0)
    lse = torch.zeros((1, g * h, w), device=DEV) if given_lse else None      # (the dominant key's logit is 0)
    got = adakv.score(layer, q, K, row_lse=lse).cpu().numpy().astype(np.float64).reshape(h, n)
    x = K[:n, :, 0].double().cpu().numpy().T
    want = np.exp(x) if given_lse else np.exp(x) / np.exp(x).sum(axis=1, keepdims=True)
    assert np.all(np.abs(got - want) <= 3e-5 * want + 2 * 2.0 ** -149)
    assert np.all(got[want > 3 * 2.0 ** -149] > 0)


@pytest.mark.parametrize("w", [5, 16, 33])             # 10, 32 and 66 window rows
def test_an_infinite_logit_gives_an_infinite_score(w):
    """With the caller's log-sum-exp one infinite key is its own affair: an infinite weight in every row,
    whether or not the rows fill their blocks of 32, and finite scores elsewhere."""
    print("fp32 infinite logit", w, flush=True)
    h, g, d, n = 2, 2, 64, 200
    wl = synth.small_workload(g * h, h, d, w, 1, [n], [h * w], dtype=torch.float32, seed=3, temps=(0.25, 1.0))
    q, K, _ = synth.generate(wl, device=DEV)
    q[..., 0] = q[..., 0].abs() + 0.1
    lse = synth.prefill_row_lse(wl, q, K)
    layer = adakv.Layer.from_workload(wl)
    clean = adakv.score(layer, q, K, row_lse=lse).reshape(h, n)
    K[77, :, 0] = float("inf")
    got = adakv.score(layer, q, K, row_lse=lse).reshape(h, n)
    assert torch.all(got[:, 77] == float("inf"))
    got[:, 77] = clean[:, 77]
    assert torch.equal(got, clean)


@pytest.mark.parametrize("k", [1, 7, 33, 35])          # no pool; in the sweep (radius 3, 16); in a kernel of its own
@pytest.mark.parametrize("n", [[3, 40], [122, 129, 300]])
def test_a_key_that_is_not_a_number_shows_in_every_score(k, n):
    """A NaN key makes every row's log-sum-exp, and so every weight of its head, a NaN; the scores say so up
    to the ends of the sequence, and the other heads are left alone."""
    print("fp32 nan key", k, n, flush=True)
    wl = synth.small_workload(4, 2, 64, 8, k, n, [2 * 8] * len(n), dtype=torch.float32, seed=5)
    q, K, _ = synth.generate(wl, device=DEV)
    layer = adakv.Layer.from_workload(wl)
    clean = adakv.score(layer, q, K)
    for b, nb in enumerate(n):
        K[wl.tok_off[b] + nb // 2, 1, 5] = float("nan")
    got, at = adakv.score(layer, q, K), 0
    for nb in n:
        assert torch.equal(got[at:at + nb], clean[at:at + nb])
        assert torch.isnan(got[at + nb:at + 2 * nb]).all(), nb
        at += 2 * nb
