"""fp32 scoring with products made of bf16 parts: every one of the products, row blocks of 32 with remainders, more rows
than the weights sweep keeps log-sum-exps of (2048), values at the ends of the parts' range, and those that take the
fp32 instruction."""
import numpy as np
import pytest
import torch

import paper_2407_11550_amd as adakv
from paper_2407_11550_amd import synth
from test_gpu_score_f32 import DEV, _reference

pytestmark = pytest.mark.gpu


def _cut(layer):
    """The layer, which has to be one that is scored with products of parts."""
    desc = adakv.describe(layer)
    assert (desc["score"], desc["products"]) == ("fma", "parts")
    return layer


def _compare(h_q, h, d, w, k, n, given_lse, change=None, visible=()):
    """visible: columns without each of which scores would be off by far more than the tolerance."""
    print("parts", h_q, h, d, w, k, n, given_lse, flush=True)
    wl = synth.small_workload(h_q, h, d, w, k, n, [h * w] * len(n), dtype=torch.float32, seed=17, temps=(0.25, 1.0))
    q, K, _ = synth.generate(wl, device=DEV)
    if change:
        change(q, K)
    lse = synth.prefill_row_lse(wl, q, K) if given_lse else None
    got = adakv.score(_cut(adakv.Layer.from_workload(wl)), q, K, row_lse=lse).cpu().numpy().astype(np.float64)
    want, tol = _reference(wl, q, K, lse)      # d roundings of a logit at the size of its products' magnitudes
    assert tol < 2e-3
    err = np.abs(got - want) / want
    assert err.max() <= tol, (err.max(), tol)
    for column in visible:
        q0 = q.clone()
        q0[..., column] = 0.0
        assert (np.abs(_reference(wl, q0, K, lse)[0] - want) / want).max() > 100 * tol


EDGES = [
    (2, 2, 128, 33, [31, 300]),                # a row block and one row
    (4, 2, 128, 32, [129, 4097]),              # two whole ones; statistics combined by a kernel
    (10, 2, 64, 13, [128, 1]),                 # d = 64: 65 rows
    (4, 2, 64, 33, [33, 4100]),                # 66; statistics combined by a kernel
    (16, 8, 128, 32, [5000]),                  # statistics per 256 keys, combined in the sweep
    (16, 8, 64, 33, [5001]),
    (64, 1, 128, 32, [200]),                   # 2048 rows, all log-sum-exps at once
    (64, 1, 64, 33, [140]),                    # 2112: a second lot
]


@pytest.mark.parametrize("given_lse", [False, True], ids=["sweep", "row_lse"])
@pytest.mark.parametrize("h_q,h,d,w,n", EDGES)
def test_edges(h_q, h, d, w, n, given_lse):
    _compare(h_q, h, d, w, 7, n, given_lse)


@pytest.mark.parametrize("q_val,k_val", [
    (2.0 ** -57, 2.0 ** 59.9),                 # the largest keys that are cut
    (2.0 ** 59.9, 2.0 ** -57),                 # ... and rows
    (2.0 ** -57.5, 2.0 ** 60.5),               # keys by the fp32 instruction
    (2.0 ** 61.0, 2.0 ** -58),                 # rows by it
    (3.3e38, 2.0 ** -126.5),                   # rounds to an infinite bf16 value; subnormal keys
])
@pytest.mark.parametrize("both", [False, True], ids=["", "keys_and_rows"])
@pytest.mark.parametrize("d,w", [(128, 40), (64, 33)])
def test_ends_of_the_range(d, w, both, q_val, k_val):
    """Some rows' and keys' values in one column are as large or small as given (`both`: other keys' and rows' in another
    column the other way round); their products are 3 to 8, so that logits stay of ordinary size and scores show it if
    the column, or one of the other keys or rows, took its place."""
    def change(q, K):
        q[..., 5] = K[..., 5] = q[..., 41] = K[..., 41] = 0.0
        q[:, :, 3::7, 5] = q_val * (1 + 2.0 ** -20)
        K[2::9, :, 5] = k_val * (1 + 2.0 ** -21)
        if both:
            q[:, :, 1::5, 41] = k_val * (1 + 2.0 ** -21)
            K[4::9, :, 41] = q_val * (1 + 2.0 ** -20)
    _compare(4, 2, d, w, 1, [300], False, change, visible=[5, 41] if both else [5])


# (part of a key's value, part of a row's): what score_cut_kernel multiplies beside the first parts of both
PRODUCTS = [(0, 1), (1, 0), (0, 2), (2, 0), (1, 1)]


def products_inputs(h, d, w, n):
    """Window rows [h, w, d] and keys [n, h, d] (float64, all values exact in fp32) whose logits at scale 1, -4 to 8, are
    one product of parts each: row r has kind r % 5 and three columns of its own, in which everything else cancels.
    All products and sums are exact in fp32, in any order."""
    q, K = np.zeros((h, w, d)), np.zeros((n, h, d))
    j, c, steps = np.arange(n)[:, None], np.arange(h)[None], d // 16
    for s in range(steps):
        few = 0.25 * ((3 * j + 5 * s + 7 * c) % 16)            # 0 to 3.75
        for t, (pk, pq) in enumerate(PRODUCTS):
            at = 16 * s + 3 * t
            rows = [r for r in range(w) if r % 5 == t and r // 5 % steps == s]
            one = 1.0 + 0.25 * (np.arange(h)[:, None] + np.array(rows)[None]) % 1.0
            high = {1: 1024.0, 2: 2.0 ** 18 + 2.0 ** 9}        # what precedes a second and a third part
            if pk == 0:                                        # k (high + part) - k high
                K[..., at] = few - 2.0
                K[..., at + 1] = few - 2.0
                q[:, rows, at] = high[pq] + one
                q[:, rows, at + 1] = -high[pq]
            elif pq == 0:
                part = few if pk == 1 else few % 1.75
                K[..., at] = high[pk] + part
                K[..., at + 1] = -high[pk]
                q[:, rows, at] = one
                q[:, rows, at + 1] = one
            else:                                              # (h + m) (h' + m') - h (h' + m') - m h'
                K[..., at] = 1024.0 + few
                K[..., at + 1] = -1024.0
                K[..., at + 2] = -few
                q[:, rows, at] = 1024.0 + one
                q[:, rows, at + 1] = 1024.0 + one
                q[:, rows, at + 2] = 1024.0
    return q, K


def products_scores(logit, lse):
    """[h, w, n] -> [h, n]; and the bound: exponents below 32 have units of 2^-19, one for the logarithm and half of one
    for the scaled logit, the log-sum-exp and their difference each; 1e-6 for the exponential and the sums."""
    z = np.log(np.exp(logit).sum(axis=-1, keepdims=True)) if lse is None else lse
    assert np.abs((logit - z) / np.log(2)).max() < 32
    return np.exp(logit - z).mean(axis=1), 2.5 * 2.0 ** -19 * np.log(2) + 1e-6


@pytest.mark.parametrize("given_lse", [False, True], ids=["sweep", "row_lse"])
@pytest.mark.parametrize("d,w,n", [(128, 80, 300), (64, 65, 5000)])
def test_every_product_of_parts(d, w, n, given_lse):
    print("parts one by one", d, w, n, given_lse, flush=True)
    h = 2
    q, K = products_inputs(h, d, w, n)
    layer = _cut(adakv.Layer(torch.float32, h, h, d, w, 1, 0.2, [n], [h * w], scale=1.0))
    qt = torch.from_numpy(q).float().to(DEV)[None].contiguous()
    Kt = torch.zeros((n + w, h, d), device=DEV)
    Kt[:n] = torch.from_numpy(K).float()
    lse = torch.full((1, h, w), 4.0, device=DEV) if given_lse else None
    got = adakv.score(layer, qt, Kt, row_lse=lse).cpu().numpy().astype(np.float64).reshape(h, n)
    want, tol = products_scores(np.stack([q[c] @ K[:, c].T for c in range(h)]), 4.0 if given_lse else None)
    assert np.all(np.abs(got - want) <= tol * want), (np.abs(got / want - 1).max(), tol)


def test_an_infinite_row_is_its_own_affair():
    """-inf in one window row's query meets positive keys: that row's logits are -inf for the caller's finite
    log-sum-exp, its weights zero; the other rows' weights are what they are without it."""
    h, d, w, n = 1, 128, 48, 200
    wl = synth.small_workload(h, h, d, w, 1, [n], [h * w], dtype=torch.float32, seed=3, temps=(0.25, 1.0))
    q, K, _ = synth.generate(wl, device=DEV)
    K[..., 7] = K[..., 7].abs() + 0.1
    lse = synth.prefill_row_lse(wl, q, K)
    q[0, 0, 35, 7] = -float("inf")
    got = adakv.score(_cut(adakv.Layer.from_workload(wl)), q, K, row_lse=lse).double().cpu()
    keep = [r for r in range(w) if r != 35]
    logit = q[0, 0, keep].double().cpu() @ K[:n, 0].double().cpu().t() / d ** 0.5
    want = torch.exp(logit - lse[0, 0, keep].double().cpu()[:, None]).sum(dim=0) / w
    assert torch.all((got - want).abs() <= 1e-4 * want)


@pytest.mark.parametrize("given_lse", [False, True], ids=["sweep", "row_lse"])
@pytest.mark.parametrize("d,w", [(128, 40), (64, 70)])
def test_a_scale_that_makes_small_values_count(d, w, given_lse):
    """Logits of 0 to 63/64 out of keys near 2^-120 and a scale of 2^127: what tells the keys apart are multiples of
    2^-137, which no bf16 number holds.  Every product and sum of a logit is exact in fp32.  An exponent is below 16, with
    units of 2^-20: one for the logarithm, half of one for the scaled logit, the log-sum-exp and their difference each,
    and 1e-6 for the exponential and the sums."""
    print("parts small values", d, w, given_lse, flush=True)
    h, n = 2, 300
    t = (torch.arange((n + w) * h, device=DEV).reshape(n + w, h) * 5 % 64).double()
    K = torch.zeros((n + w, h, d), device=DEV)
    K[..., 6] = (2.0 ** -120 * (1 + t * 2.0 ** -17)).float()
    K[..., 40] = 2.0 ** -120
    q = torch.zeros((1, h, w, d), device=DEV)
    q[..., 6], q[..., 40] = 16.0, -16.0
    layer = adakv.Layer(torch.float32, h, h, d, w, 1, 0.2, [n], [h * w], scale=2.0 ** 127)
    x = (t[:n] / 64).cpu().numpy().T
    lse = torch.full((1, h, w), 2.0, device=DEV) if given_lse else None
    got = adakv.score(layer, q, K, row_lse=lse).cpu().numpy().astype(np.float64).reshape(h, n)
    want = np.exp(x - 2) if given_lse else np.exp(x) / np.exp(x).sum(axis=1, keepdims=True)
    assert np.all(np.abs(got - want) <= (2.5 * 2.0 ** -20 * np.log(2) + 1e-6) * want)
