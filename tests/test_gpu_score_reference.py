"""The statistics sweeps of the 16-bit scoring kernels keep the reference of a row that their first tile gave it.  Here
every workgroup's (up to 128 rows: wavefront's) first tiles lie far below one key further on: by so little that the sum
stays finite, where the row's log-sum-exp must not be rounded at the size of the gap, and by more than fp32 holds."""
import pytest
import torch

import paper_2407_11550_amd as adakv

DEV = "cuda:0"
TILE = 32

# h_q, h_kv, d, w, n, dtype, tiles of a set (0: every wavefront takes tiles of its own)
CASES = [
    (64, 64, 128, 1, 2511, torch.bfloat16, 0),          # one row
    (128, 64, 64, 32, 5001, torch.float16, 0),          # 64 rows, d = 64
    (256, 64, 128, 32, 2560, torch.bfloat16, 0),        # 128 rows, full tiles only
    (256, 64, 64, 31, 4703, torch.bfloat16, 0),         # 124 rows
    (512, 64, 128, 32, 1500, torch.bfloat16, 4),        # 256 rows
    (512, 64, 128, 31, 1260, torch.float16, 2),
    (512, 64, 64, 32, 619, torch.bfloat16, 2),
    (1024, 64, 128, 32, 1500, torch.bfloat16, 4),       # 512 rows
    (1024, 64, 128, 31, 1250, torch.bfloat16, 2),
    (1024, 64, 64, 32, 1501, torch.float16, 4),         # 512 rows, d = 64
    (1024, 64, 64, 32, 640, torch.bfloat16, 2),
]
IDS = ["hq%d_d%d_w%d_n%d" % (c[0], c[2], c[3], c[4]) for c in CASES]


def _layer(case):
    h_q, h, d, w, n, dt, _ = case
    return adakv.Layer(dt, h_q, h, d, w, 7, 0.2, [n], [h * w])


def _split(case):
    """(workgroups of a head, tiles that come first in one of them or of their wavefronts, the fewest full tiles that
    one of those takes), by the kernels' rules on the keys per workgroup that the library reports."""
    n, sets = case[4], case[6]
    keys = int(adakv.describe(_layer(case))["stat_keys"])
    wgs, tiles = -(-n // keys), -(-n // TILE)
    units = wgs if sets else 4 * wgs                    # sets, or tiles, are dealt out over these
    each = max(sets, 1)
    whole = n // TILE
    taken = [sum(min(each, max(0, whole - s * each)) for s in range(u, -(-tiles // each), units)) for u in range(units)]
    return wgs, units * each, taken


@pytest.mark.parametrize("case", CASES, ids=IDS)
def test_a_reference_is_kept(case, lib):
    """Four full tiles or more, so that the reference is kept, in sets of the size that the case is there for."""
    share = int(adakv.describe(_layer(case))["stat_keys"]) // TILE
    if case[6]:
        assert case[6] == (2 if -share % 4 >= 2 and -share % 4 * 8 >= share else 4), share
    wgs, first, taken = _split(case)
    assert wgs > 1 and min(taken) >= 4, (wgs, taken)
    assert first * TILE + 64 < case[4]


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=IDS)
@pytest.mark.parametrize("low,high", [(28, 76), (92, 120)], ids=["finite", "overflow"])
def test_one_key_far_above_the_kept_reference(case, low, high):
    h_q, h, d, w, n, dt, _ = case
    print("kept reference", case, low, high, flush=True)
    layer, first = _layer(case), _split(case)[1] * TILE
    layer = adakv.Layer(dt, h_q, h, d, w, 7, 0.2, [n], [h * w], scale=0.125)
    # One row of a head looks at the keys' first elements, the others at the second (8 x scale = 1): the logits are the
    # elements themselves.  The one row's key is nobody else's, so that its score is one weight and not a sum over rows.
    head, rows = torch.arange(h, device=DEV), h_q // h * w
    q = torch.zeros((h, rows, d), dtype=dt, device=DEV)
    q[..., 1] = 8.0
    q[head, 37 * head % rows, 0], q[head, 37 * head % rows, 1] = 8.0, 0.0
    q = q.reshape(1, h_q, w, d)
    K = torch.zeros((n + w, h, d), dtype=dt, device=DEV)
    gap = low + (high - low) * head // (h - 1)          # whole, and at most 120: exact in 16 bits
    K[:first, :, 0] = -gap.to(dt)
    K[first:, :, 0] = -20.0
    K[:, :, 1] = -40.0
    at = first + 7 + (n - first - 30) * head // (h - 1)                                # full tiles and the ragged one
    K[at, head, 0] = (0.25 * (head % 5)).to(dt)
    K[at + 15, head, 1] = 0.5
    got = adakv.score(layer, q, K).double().reshape(h, n)
    a = (torch.softmax(K[:n, :, 0].double().t(), dim=1) + (rows - 1) * torch.softmax(K[:n, :, 1].double().t(), dim=1)) / rows
    want = torch.nn.functional.max_pool1d(a[None], 7, 1, 3)[0]
    err = (got - want).abs() / want
    # The one key's logit x (below 2 in base 2) is a product rounded at its size, as is the log-sum-exp, which is x + log2
    # of a sum within 1e-5 of one, and their difference: 2^-24 each, the logarithm 2^-23; times ln 2; an exponential of 1 ulp.
    # The sum itself is that key's 1 and what lanes, wavefronts and workgroups (2, 4 and at most 8) add to it, 2^-24 each.
    near = err[head, at]
    assert near.max().item() <= 0.6932 * 5 * 2.0 ** -24 + 2.0 ** -23 + 14 * 2.0 ** -24, (near.max().item(), int(near.argmax()))
    # Keys 20 below it: their logit, 29 in base 2, is rounded to 2^-20, and log2(e) to 2^-24 of it; twice that for the
    # log-sum-exp and the exponential, and 2^-24 for each of the rows added up.
    assert err[want > 1e-10 / rows].max().item() <= 2 * 0.6932 * (2.0 ** -20 + 29 * 2.0 ** -24) + rows * 2.0 ** -24
