"""Top-k scopes that run inside one block (up to 16384 scores of a sequence or of a head; 4, 12 or 16
rounds of 1024): the calls on their own and inside adakv_compress, against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import paper_2407_11550_amd as adakv
from oracle import adakv_oracle as O
from paper_2407_11550_amd import synth

from parity_util import assert_exact_on_scores

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _scores(rng, kind, h, n):
    if kind == "spread":
        return (rng.random((h, n)) ** 8).astype(np.float32)
    if kind == "pooled":
        return O.max_pool_same((rng.random((h, n)) ** 12).astype(np.float32), 7).astype(np.float32)
    if kind == "equal":
        return np.full((h, n), 0.25, np.float32)
    if kind == "zeros":                                  # underflowed weights, the budget reaches into them
        return np.where(rng.random((h, n)) < 0.02, rng.random((h, n)), 0.0).astype(np.float32)
    one = np.array([0.3], np.float32).view(np.uint32)[0] & ~np.uint32(1023)
    return (one + rng.integers(0, 1024, (h, n)).astype(np.uint32)).view(np.float32)      # one 22-bit prefix


# KV heads, prefix lengths around the rounds of 1024, the four sizes and the largest one-block scopes
LAYERS = [
    (4, [1, 2, 63, 64, 65, 1023, 1024, 1025]),
    (4, [1000, 4096, 4097, 16383, 16385]),
    (8, [2048, 2047, 5]),                      # exactly 16384 scores: a sequence in one block
    (8, [2049]),                               # one more position per head: the layer scope by the gather kernels
    (5, [16384, 31]),                          # the longest head in one block
    (5, [16385]),                              # and one past it
    (2, [40000]),                              # beyond a block in either scope
    (64, [700, 1024]),
    (16, [768]), (16, [769]),                  # 12 288 scores of more than eight heads in a block, and past it
    (64, [128, 7]), (64, [129]),               # 8192 of more than 32
    (64, [80] * 9),                            # 576 segments
]


@pytest.mark.parametrize("kind", ["spread", "pooled", "equal", "zeros", "one_prefix"])
@pytest.mark.parametrize("layer_no", range(len(LAYERS)))
def test_allocate_and_select_alone(layer_no, kind):
    h, lengths = LAYERS[layer_no]
    print("topk block", h, lengths, kind, flush=True)
    rng = np.random.default_rng(100 * layer_no + len(kind))
    w = 3
    for keep in (0.0, 0.03, 0.5, 1.0):
        B = [h * w + int(keep * h * n) for n in lengths]
        layer = adakv.Layer(torch.bfloat16, h, h, 64, w, 7, 0.2, lengths, B)
        sc = [_scores(rng, kind, h, n) for n in lengths]
        flat = torch.from_numpy(np.concatenate([s.reshape(-1) for s in sc])).to(DEV)
        bud, cu = adakv.allocate(layer, flat)
        guard = torch.full((sum(B) + 256,), -5, dtype=torch.int32, device=DEV)
        adakv.select(layer, flat, bud, cu, indices=guard)
        bud, cu, idx = bud.cpu().numpy(), cu.cpu().numpy(), guard.cpu().numpy()
        assert np.all(idx[sum(B):] == -5)
        row0 = 0
        for b, n in enumerate(lengths):
            ob, oc = O.allocate(sc[b], B[b], w, 0.2)
            assert np.array_equal(bud[b * h:(b + 1) * h], ob), (n, keep)
            assert np.array_equal(cu[b * h:(b + 1) * h + 1], oc + row0), (n, keep)
            assert np.array_equal(idx[row0:row0 + B[b]], O.select(sc[b], ob, w)), (n, keep)
            row0 += B[b]


# h_q, h_kv, d, w, n: both scopes in one launch, the head scope in one, neither
STEPS = [
    (8, 4, 128, 8, [700, 40]),
    (8, 8, 64, 4, [1536]),                     # 12288 scores: the most that run in one launch
    (8, 8, 64, 4, [1537]),                     # gather and one launch
    (4, 4, 64, 2, [4096, 4095]),               # the longest head of that form
    (4, 4, 64, 2, [4097]),
    (4, 4, 64, 2, [8192, 5]),                  # the longest head of the one-launch head scope
    (4, 4, 64, 2, [8193]),
    (32, 32, 64, 2, [70] * 17),                # 544 segments: more blocks than compute units would repeat the layer scope
    (2, 2, 64, 2, [900]),                      # two segments
    (1, 1, 64, 2, [12288, 9]),                 # one head: the most that run in one launch
    (1, 1, 64, 2, [12289]),
    (3, 3, 64, 2, [4096]),
    (2, 2, 64, 2, [8192]),                     # two kernels for the layer, one block per head
]


@pytest.mark.parametrize("keep", [0.0, 0.05, 1.0])
@pytest.mark.parametrize("step", STEPS, ids=lambda s: "h%d_n%s" % (s[1], "-".join(map(str, s[4][:3]))))
def test_whole_step(step, keep):
    h_q, h, d, w, n = step
    print("topk step", step, keep, flush=True)
    B = [h * w + int(keep * h * nb) for nb in n]
    wl = synth.small_workload(h_q, h, d, w, 7, n, B, seed=17)
    q, K, V = synth.generate(wl, device=DEV)
    layer = adakv.Layer.from_workload(wl)
    ws = torch.full((adakv.workspace_bytes(layer),), 0xAB, dtype=torch.uint8, device=DEV)
    out = adakv.compress(layer, q, K, V, ws=ws)
    sc, row0, soff = out["scores"].cpu().numpy(), 0, 0
    for b in range(wl.batch):
        assert_exact_on_scores(out, sc[soff:soff + h * n[b]], wl, K, V, b, seg0=b * h, row0=row0)
        row0 += B[b]
        soff += h * n[b]


# 32 KV heads; prefix length, sequences, the Top-k kernels of the step
MANY = [
    (70, 8, ["topk_block"]),                                  # 256 segments: one block per compute unit
    (70, 9, ["alloc_gather", "alloc_finish", "select_block"]),
    (400, 8, ["alloc_gather", "topk_block"]),                 # 12 800 scores per sequence
    (400, 9, ["alloc_gather", "alloc_finish", "select_block"]),
]


@pytest.mark.parametrize("n,nseq,kernels", MANY)
def test_no_more_repeated_layer_scopes_than_compute_units(n, nseq, kernels):
    """A block per segment that repeats the layer scope for itself only while there is a compute unit for each."""
    print("topk many segments", n, nseq, flush=True)
    h, w = 32, 2
    B = [h * w + h * n // 20] * nseq
    wl = synth.small_workload(h, h, 64, w, 7, [n] * nseq, B, seed=19)
    q, K, V = synth.generate(wl, device=DEV)
    layer = adakv.Layer.from_workload(wl)
    with adakv.KernelTrace(64) as tr:
        out = adakv.compress(layer, q, K, V)
    torch.cuda.synchronize()
    assert [k for k, _ in tr.durations_us() if k.split("_")[0] in ("topk", "alloc", "select")] == kernels
    sc = out["scores"].cpu().numpy()
    for b in range(nseq):
        assert_exact_on_scores(out, sc[b * h * n:(b + 1) * h * n], wl, K, V, b, seg0=b * h, row0=b * B[0])


@pytest.mark.parametrize("n", [600, 5000, 20000])      # both scopes in a block, the head scope, neither
def test_scores_with_all_bits_set_are_positions_like_others(n):
    """Memory that was filled with ones (a NaN, outside the contract) comes last, by position, and a budget
    that takes everything still lists every position once."""
    print("topk all bits set", n, flush=True)
    h, w = 2, 3
    bits = np.random.default_rng(n).random((h, n)).astype(np.float32).view(np.int32)
    bits[:, ::3] = -1
    flat = torch.from_numpy(bits.reshape(-1).copy()).to(DEV).view(torch.float32)
    for keep in (n, n - n // 6):
        layer = adakv.Layer(torch.bfloat16, h, h, 64, w, 7, 1.0, [n], [h * (w + keep)])
        bud, cu = adakv.allocate(layer, flat)
        assert bud.tolist() == [keep] * h
        idx = torch.full((layer.num_rows_out,), -5, dtype=torch.int32, device=DEV)
        adakv.select(layer, flat, bud, cu, indices=idx)
        numbers = [j for j in range(n) if j % 3]
        want = sorted(numbers + list(range(0, n, 3))[:keep - len(numbers)]) + list(range(n, n + w))
        assert idx.cpu().tolist() == want * h


@pytest.mark.parametrize("h,n,block", [(8, 2048, True), (8, 2049, False), (9, 1365, True), (9, 1366, False),
                                       (32, 384, True), (32, 385, False), (33, 248, True), (33, 249, False)])
def test_one_block_allocates_fewer_scores_the_more_heads_there_are(h, n, block):
    print("alloc route", h, n, flush=True)
    layer = adakv.Layer(torch.bfloat16, h, h, 64, 3, 7, 0.2, [n], [h * (3 + n // 9)])
    scores = torch.rand(h * n, device=DEV)
    with adakv.KernelTrace(16) as tr:
        bud, _ = adakv.allocate(layer, scores)
    torch.cuda.synchronize()
    assert [k for k, _ in tr.durations_us()] == (["alloc_block"] if block else
                                                 ["alloc_init", "alloc_pass0", "alloc_gather", "alloc_finish"])
    want, _ = O.allocate(scores.cpu().numpy().reshape(h, n), layer.B[0], 3, 0.2)
    assert np.array_equal(bud.cpu().numpy(), want)
