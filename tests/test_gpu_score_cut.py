"""fp32 scoring with products made of bf16 parts: row blocks of 32 with remainders, more rows than the weights sweep
keeps log-sum-exps of (2048), values at the ends of the parts' range, and those that take the fp32 instruction."""
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


def _compare(h_q, h, d, w, k, n, given_lse, change=None):
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
    (2.0 ** -70, 2.0 ** 59.9),                 # the largest that are cut
    (2.0 ** -70, 2.0 ** 60.5),                 # keys by the fp32 instruction
    (2.0 ** 61.0, 2.0 ** -75),                 # rows by it
    (2.0 ** 50.0, 2.0 ** -126),                # the keys' last parts lie below bf16's normal range
    (3.3e38, 2.0 ** -132),                     # rounds to an infinite bf16 value; subnormal keys
])
@pytest.mark.parametrize("d,w", [(128, 40), (64, 33)])
def test_ends_of_the_range(d, w, q_val, k_val):
    """Some keys' (rows') values in one column are as large or small as given; all logits stay of ordinary size."""
    def change(q, K):
        q[..., 5] = 0.0
        K[..., 5] = 0.0
        q[:, :, 3::7, 5] = q_val * (1 + 2.0 ** -20)
        K[2::9, :, 5] = k_val * (1 + 2.0 ** -21)
    _compare(4, 2, d, w, 1, [300], False, change)


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
