"""CPU-side check of what test_gpu_score_cut.py can see: with fp32 values cut into three bf16 parts as the kernel cuts
them, the six products that it takes give the test's scores, and no five of them do."""
import numpy as np
import pytest

from test_gpu_score_cut import PRODUCTS, products_inputs, products_scores

TAKEN = PRODUCTS + [(0, 0)]


def _bf16(x):
    """Rounded to nearest, ties to even."""
    bits = np.ascontiguousarray(x, dtype=np.float32).view(np.uint32)
    return ((bits + 0x7FFF + (bits >> 16 & 1)) & np.uint32(0xFFFF0000)).view(np.float32)


def _parts(x):
    rest, out = x.astype(np.float32), []
    assert np.array_equal(rest.astype(np.float64), x)
    for _ in range(3):
        out.append(_bf16(rest))
        rest = rest - out[-1]
    assert not rest.any()
    return [p.astype(np.float64) for p in out]


def _scores(q, K, taken, lse):
    logit = np.zeros((q.shape[0], q.shape[1], K.shape[0]))
    for c in range(q.shape[0]):
        qp, kp = _parts(q[c]), _parts(K[:, c])
        for pk, pq in taken:
            logit[c] += qp[pq] @ kp[pk].T
    z = np.log(np.exp(logit - logit.max()).sum(axis=-1, keepdims=True)) + logit.max() if lse is None else lse
    return np.exp(logit - z).mean(axis=1)


@pytest.mark.parametrize("lse", [None, 4.0], ids=["sweep", "row_lse"])
@pytest.mark.parametrize("d,w", [(128, 80), (64, 65)])
def test_a_lost_product_shows(d, w, lse):
    q, K = products_inputs(2, d, w, 300)
    logit = np.stack([q[c] @ K[:, c].T for c in range(2)])
    assert logit.min() >= -4 and logit.max() <= 8
    want, tol = products_scores(logit, lse)
    assert np.abs(_scores(q, K, TAKEN, lse) / want - 1).max() < 1e-12
    with np.errstate(all="ignore"):
        for lost in TAKEN:
            off = np.abs(_scores(q, K, [p for p in TAKEN if p != lost], lse) / want - 1).max()
            assert not off <= 1000 * tol, lost
        for a, b in ((1, 2), (0, 1)):                      # parts taken for each other
            mixed = [tuple({a: b, b: a}.get(x, x) if i == 0 else x for i, x in enumerate(p)) for p in TAKEN]
            assert not np.abs(_scores(q, K, mixed, lse) / want - 1).max() <= 1000 * tol
