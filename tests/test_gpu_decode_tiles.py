"""Decode attention on 16-bit caches at the edges of its split: tiles of 32 rows, four wavefronts of
one tile each per round, workgroups of 64 rows or a multiple of 128, or of eight wavefronts over a
whole short segment; an appended row in the last
place of a tile or the first of a new one; and values at the ends of the types' ranges."""
import numpy as np
import pytest
import torch

import paper_2407_11550_amd as adakv
from oracle import decode_oracle as D
from paper_2407_11550_amd import synth

from parity_util import to_f64
from test_gpu_decode import _assert_decode_close

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
LENGTHS = [1, 2, 15, 16, 31, 32, 33, 63, 64, 65, 95, 127, 128, 129, 192, 193]


def _cache(dt, d, g, lengths, headroom, seed):
    h, w = len(lengths), 1
    n = max(lengths) + 7
    wl = synth.small_workload(g * h, h, d, w, 7, [n], [sum(lengths)], dtype=dt, seed=seed)
    Kc, Vc, cu, lens = synth.ragged_cache(wl, [v - w for v in lengths], headroom, seed=seed, device=DEV)
    for s in range(h):                                   # spare rows must never be read
        a = int(cu[s + 1]) + s * headroom
        Kc[a:a + headroom] = float("nan")
        Vc[a:a + headroom] = float("nan")
    return wl, adakv.Layer.from_workload(wl), Kc, Vc, cu, lens


@pytest.mark.parametrize("g", [1, 2, 4, 8])
@pytest.mark.parametrize("dt,d", [(torch.bfloat16, 128), (torch.bfloat16, 64), (torch.float16, 128), (torch.float16, 64)])
# more rows per segment: one workgroup per segment, splits of 64 rows, splits of a multiple of 128
@pytest.mark.parametrize("longer", [0, 400, 9000], ids=["whole", "rows64", "rows128"])
def test_decode_step_at_tile_edges(dt, d, g, longer):
    print("decode tiles", dt, d, g, longer, flush=True)
    lengths = [v + longer for v in LENGTHS]
    hr = 2
    wl, layer, Kc, Vc, cu, lens = _cache(dt, d, g, lengths, hr, seed=40 + g)
    q, kn, vn = synth.decode_inputs(wl, 2, seed=g, device=DEV)
    oK, oV = to_f64(Kc), to_f64(Vc)
    olen, cuh = lens.cpu().numpy().astype(np.int64), cu.cpu().numpy()
    vmax = float(torch.nan_to_num(Vc.float(), nan=0.0).abs().max())
    for t in range(2):
        out, lse = adakv.decode_step(layer, q[t], kn[t], vn[t], cu, hr, Kc, Vc, lens, want_lse=True)
        torch.cuda.synchronize()
        D.append(oK, oV, cuh, hr, olen, to_f64(kn[t]).reshape(-1, d), to_f64(vn[t]).reshape(-1, d))
        assert np.array_equal(lens.cpu().numpy(), olen)
        ref_out, ref_lse = D.decode_attention(to_f64(q[t]), oK, oV, cuh, hr, olen, wl.g)
        _assert_decode_close(out, lse, ref_out, ref_lse, vmax, f"step {t}")
        assert np.array_equal(to_f64(Kc), oK, equal_nan=True) and np.array_equal(to_f64(Vc), oV, equal_nan=True)
    full = torch.zeros(1, dtype=torch.int32, device=DEV)                  # no room left: nothing appended, and said so
    before = [t.clone() for t in (Kc, Vc, lens)]
    out, lse = adakv.decode_step(layer, q[0], kn[0], vn[0], cu, hr, Kc, Vc, lens, overflow=full, want_lse=True)
    ref_out, ref_lse = D.decode_attention(to_f64(q[0]), oK, oV, cuh, hr, olen, wl.g)
    _assert_decode_close(out, lse, ref_out, ref_lse, vmax, "full")
    assert int(full) == 1
    assert all(torch.equal(torch.nan_to_num(a.float()), torch.nan_to_num(b.float())) for a, b in zip(before, (Kc, Vc, lens)))


@pytest.mark.parametrize("g", [4, 8])
@pytest.mark.parametrize("dt,tiny", [(torch.float16, 2.0 ** -18), (torch.bfloat16, 2.0 ** -100)], ids=["fp16", "bf16"])
def test_decode_values_at_the_ends_of_the_range(dt, tiny, g):
    """fp16 values below the normal range keep their bits, and an infinite value row gives the
    infinity (not the NaN that 0 * inf of a cut weight would make)."""
    print("decode range", dt, g, flush=True)
    wl, layer, Kc, Vc, cu, lens = _cache(dt, 128, g, [300, 77], 1, seed=3)
    q, _, _ = synth.decode_inputs(wl, 1, seed=3, device=DEV)
    Vt = (Vc.float() * tiny).to(dt)
    out = adakv.decode_attn(layer, q[0], cu, 1, Kc, Vt, lens)
    ref, _ = D.decode_attention(to_f64(q[0]), to_f64(Kc), to_f64(Vt), cu.cpu().numpy(), 1, lens.cpu().numpy(), g)
    _assert_decode_close(out / tiny, None, ref / tiny, None, float(torch.nan_to_num(Vc.float(), nan=0.0).abs().max()), "tiny")
    Vi = Vc.clone()
    Vi[5, 17] = float("inf")
    Vi[6, 18] = float("-inf")
    got = adakv.decode_attn(layer, q[0], cu, 1, Kc, Vi, lens)[0, :g].cpu()
    assert torch.all(got[:, 17] == float("inf")) and torch.all(got[:, 18] == float("-inf"))
    keep = [e for e in range(128) if e not in (17, 18)]
    assert torch.isfinite(got[:, keep]).all()


@pytest.mark.parametrize("longer", [0, 900], ids=["whole", "split"])
@pytest.mark.parametrize("g", [1, 4, 8])
@pytest.mark.parametrize("dt,d", [(torch.float16, 64), (torch.float16, 128), (torch.bfloat16, 128)])
def test_decode_small_weights_keep_their_bits(dt, d, g, longer):
    """Rows far below the maximum of their tile (2^-11 to 2^-109 of it) decide the result where the rows
    at the maximum hold zeros: every weight has 24 bits, and an infinite value behind a small one still
    gives the infinity.  Bound: a weight is exp2 of an exponent of up to 110 that was rounded to 2^-24 of
    itself three times (logit, scaling, maximum), 110 ln 2 * 3 * 2^-24 = 1.4e-5 of it, and some 2^-22 for
    the sums; stated against the sum of |weight * value|."""
    levels = [8.0, 14.0, 20.0, 30.0, 45.0, 70.0]
    print("decode small weights", dt, d, g, longer, flush=True)
    wl, _, Kc, Vc, cu, lens = _cache(dt, d, g, [97 + longer + 5 * i for i in range(len(levels))], 1, seed=9)
    layer = adakv.Layer(dt, wl.h_q, wl.h_kv, d, wl.w, 7, 0.2, wl.n, wl.B, scale=1.0)
    q = torch.zeros((1, wl.h_q, d), dtype=dt, device=DEV)
    q[:, :, 0] = 1.0
    q[:, 1::2, 0] = 0.75
    for s, level in enumerate(levels):
        a, L = int(cu[s]) + s, int(lens[s])
        r = torch.arange(L, device=DEV)
        Kc[a:a + L, 0] = torch.where(r % 16 == 0, 0.0, -(level + 0.25 * (r % 7))).to(dt)
        Vc[a:a + L] = torch.where((r % 16 == 0)[:, None], 0.0, 100.0 * Vc[a:a + L].float()).to(dt)
    out, lse = adakv.decode_attn(layer, q, cu, 1, Kc, Vc, lens, want_lse=True)
    args = (cu.cpu().numpy(), 1, lens.cpu().numpy(), g)
    ref, ref_lse = D.decode_attention(to_f64(q), to_f64(Kc), to_f64(Vc), *args, scale=1.0)
    mass, _ = D.decode_attention(to_f64(q), to_f64(Kc), np.abs(to_f64(Vc)), *args, scale=1.0)
    err = np.abs(to_f64(out) - ref) / mass
    print("  worst error", err.max(), flush=True)
    assert err.max() <= 2e-5
    assert np.abs(to_f64(lse) - ref_lse).max() <= 2e-5
    s = levels.index(30.0)
    a = int(cu[s]) + s
    Vc[a + 5, 7], Vc[a + 38, 8] = float("inf"), float("-inf")
    got = adakv.decode_attn(layer, q, cu, 1, Kc, Vc, lens)[0, s * g:(s + 1) * g].cpu()
    assert torch.all(got[:, 7] == float("inf")) and torch.all(got[:, 8] == float("-inf"))
    assert torch.isfinite(got[:, [e for e in range(d) if e not in (7, 8)]]).all()


@pytest.mark.parametrize("longer", [0, 900], ids=["whole", "split"])
@pytest.mark.parametrize("g", [1, 2, 8])
@pytest.mark.parametrize("dt,d", [(torch.float16, 64), (torch.bfloat16, 128), (torch.float32, 128)])
def test_decode_infinite_value_in_the_last_row(dt, d, g, longer):
    """The last row of a segment, held or appended by the call, is repeated in the places behind it when a
    tile is not full; an infinite value there gives the infinity in its column and touches no other."""
    print("decode last row", dt, d, g, longer, flush=True)
    lengths = [longer + v for v in (1, 2, 17, 31, 33, 45, 64, 96)]
    _, layer, Kc, Vc, cu, lens = _cache(dt, d, g, lengths, 1, seed=21)
    q, kn, vn = synth.decode_inputs(synth.small_workload(g * len(lengths), len(lengths), d, 1, 7, [8], [len(lengths)], dtype=dt, seed=21),
                                    1, seed=21, device=DEV)
    rest = [e for e in range(d) if e not in (3, 4)]
    for s in range(len(lengths)):
        a = int(cu[s]) + s + lengths[s] - 1
        Vc[a, 3], Vc[a, 4] = float("inf"), float("-inf")
    out = adakv.decode_attn(layer, q[0], cu, 1, Kc, Vc, lens).cpu()
    assert torch.all(out[..., 3] == float("inf")) and torch.all(out[..., 4] == float("-inf"))
    assert torch.isfinite(out[..., rest]).all()
    Vc[torch.isinf(Vc)] = 0.0
    vn[0, ..., 3], vn[0, ..., 4] = float("inf"), float("-inf")
    out = adakv.decode_step(layer, q[0], kn[0], vn[0], cu, 1, Kc, Vc, lens).cpu()
    assert torch.all(out[..., 3] == float("inf")) and torch.all(out[..., 4] == float("-inf"))
    assert torch.isfinite(out[..., rest]).all()


# per sequence the rows of its heads; head-room; head dimension; one workgroup per segment
ROUTES = [
    ([[64] * 4], 256, 128, True),
    ([[2040, 8, 8, 8]] + [[50] * 4] * 7, 16, 128, False),     # short on average, one long segment
    ([[500] * 4] + [[20] * 4] * 7, 16, 128, False),           # one sequence whose heads may be long
    ([[464, 100, 100, 100]], 16, 128, True),                  # 748 + 4 + 16 rows at most
    ([[465, 100, 100, 100]], 16, 128, False),                 # four times the average: one more
    ([[465, 100, 100, 100]], 16, 64, True),                   # half the bytes
    ([[460, 71] + [72] * 6], 89, 128, True),                  # eight heads: four times the average 561, at most 931 + 4 + 89 rows
    ([[460] + [72] * 7], 89, 128, False),                     # one more
    ([[460] + [72] * 7], 89, 64, True),
    ([[128] * 4], 256, 128, True),
    ([[129] * 4], 256, 128, False),                           # more than 384 rows of capacity on average
]


@pytest.mark.parametrize("rows,hr,d,whole", ROUTES)
def test_one_workgroup_per_segment_only_where_no_segment_can_be_long(rows, hr, d, whole):
    h, g, w = len(rows[0]), 2, 4
    print("decode routes", rows[0], len(rows), hr, d, flush=True)
    wl = synth.small_workload(g * h, h, d, w, 7, [4000] * len(rows), [sum(r) for r in rows], dtype=torch.bfloat16, seed=5)
    layer = adakv.Layer.from_workload(wl)
    Kc, Vc, cu, lens = synth.ragged_cache(wl, [v - w for r in rows for v in r], hr, seed=5, device=DEV)
    q, kn, vn = synth.decode_inputs(wl, 1, seed=5, device=DEV)
    with adakv.KernelTrace(16) as tr:
        out, lse = adakv.decode_step(layer, q[0], kn[0], vn[0], cu, hr, Kc, Vc, lens, want_lse=True)
    torch.cuda.synchronize()
    assert [n for n, _ in tr.durations_us()] == ["decode_attn"] + ([] if whole else ["decode_combine"])
    ref_out, ref_lse = D.decode_attention(to_f64(q[0]), to_f64(Kc), to_f64(Vc), cu.cpu().numpy(), hr, lens.cpu().numpy(), g)
    _assert_decode_close(out, lse, ref_out, ref_lse, float(Vc.float().abs().max()), f"{rows[0]}")
