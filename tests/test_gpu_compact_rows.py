"""The gather with two rows per lane group (more than 2048 blocks of rows): segments of any length
inside a block, the last block ragged, both layouts, against plain indexing, byte for byte."""
import numpy as np
import pytest
import torch

import paper_2407_11550_amd as adakv

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("headroom", [None, 3], ids=["compact", "cache_build"])
@pytest.mark.parametrize("dt,d", [(torch.bfloat16, 64), (torch.float16, 128), (torch.float32, 128)])
@pytest.mark.parametrize("extra", [0, 1, 37], ids=lambda e: "plus%d" % e)
def test_many_rows(dt, d, headroom, extra):
    print("compact rows", dt, d, headroom, extra, flush=True)
    lpr = d * (4 if dt == torch.float32 else 2) // 16
    total = 2048 * (256 // lpr) + extra                      # at and just past the line
    h, w, batch = 8, 1, 9
    nseg = h * batch
    rng = np.random.default_rng(d + extra)
    lens = np.full(nseg, w, np.int64)                        # many one-row segments, some of a block's size, a few huge
    lens[rng.choice(nseg, 20, replace=False)] += rng.integers(1, 40, 20)
    lens[::7] += (total - lens.sum()) // len(lens[::7])
    lens[0] += total - lens.sum()
    assert lens.sum() == total and lens.min() >= w
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    n = [int(lens.max()) + 11 * b for b in range(batch)]
    B = [int(lens[b * h:(b + 1) * h].sum()) for b in range(batch)]
    layer = adakv.Layer(dt, h, h, d, w, 7, 0.2, n, B)
    g = torch.Generator(device=DEV)
    g.manual_seed(5)
    rows = layer.last_token_row
    K = torch.randn((rows, h, d), generator=g, device=DEV).to(dt)
    V = torch.randn((rows, h, d), generator=g, device=DEV).to(dt)
    off, idx, src, head = layer.tok_off, [], [], []
    for s in range(nseg):
        at = rng.integers(0, n[s // h] + w, lens[s])
        idx.append(at)
        src.append(at + off[s // h])
        head.append(np.full(lens[s], s % h))
    pick = (torch.from_numpy(np.concatenate(src)).to(DEV), torch.from_numpy(np.concatenate(head)).to(DEV))
    idx_t = torch.from_numpy(np.concatenate(idx).astype(np.int32)).to(DEV)
    cu_t = torch.from_numpy(cu).to(DEV)
    if headroom is None:
        Ko, Vo = adakv.compact(layer, K, V, idx_t, cu_t)
        assert torch.equal(Ko, K[pick]) and torch.equal(Vo, V[pick])
        return
    Kc = torch.full((adakv.cache_rows(layer, headroom), d), -9.0, dtype=dt, device=DEV)
    Vc = Kc.clone()
    _, _, seg_len = adakv.cache_build(layer, K, V, idx_t, cu_t, headroom, Kc, Vc)
    place = torch.from_numpy(np.arange(total) + np.repeat(np.arange(nseg), lens) * headroom).to(DEV)
    wantK, wantV = torch.full_like(Kc, -9.0), torch.full_like(Vc, -9.0)
    wantK[place], wantV[place] = K[pick], V[pick]
    assert torch.equal(Kc, wantK) and torch.equal(Vc, wantV)
    assert np.array_equal(seg_len.cpu().numpy(), lens)
