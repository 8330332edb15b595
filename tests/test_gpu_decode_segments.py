"""How a decoding step's workgroups find their rows, up to 64 segments a lane each in every wavefront and beyond them
through LDS, and how many partial results the merge kernel has to look at: none, one, and more than it has places for."""
import numpy as np
import pytest
import torch

import paper_2407_11550_amd as adakv
from oracle import decode_oracle as D
from paper_2407_11550_amd import synth

from parity_util import to_f64
from test_gpu_decode import DEV, _assert_decode_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,h,longest", [(1, 1, 9000), (7, 9, 700), (8, 8, 700), (5, 13, 700), (2, 40, 2000)])
@pytest.mark.parametrize("dt,g,d", [(torch.bfloat16, 4, 128), (torch.float16, 8, 64), (torch.float32, 2, 64), (torch.bfloat16, 1, 128)])
def test_step_over_uneven_segments(batch, h, longest, dt, g, d):
    print("decode segments", batch, h, longest, dt, g, d, flush=True)
    rng, w, hr = np.random.default_rng(batch * h), 1, 2
    rows = rng.integers(1, longest, (batch, h))
    rows[0, 0] = longest
    n = [longest] * batch
    wl = synth.small_workload(g * h, h, d, w, 7, n, [int(r.sum()) for r in rows], dtype=dt, seed=9)
    Kc, Vc, cu, lens = synth.ragged_cache(wl, [int(v) - w for v in rows.reshape(-1)], hr, seed=9, device=DEV)
    if batch * h > 1:
        lens[-1] = 0                                     # an empty segment, and one without room
    lens[0] += hr
    Kc, Vc = torch.nan_to_num(Kc.float(), nan=0.0).to(dt), torch.nan_to_num(Vc.float(), nan=0.0).to(dt)
    q, kn, vn = synth.decode_inputs(wl, 1, seed=2, device=DEV)
    oK, oV, cuh, olen = to_f64(Kc), to_f64(Vc), cu.cpu().numpy(), lens.cpu().numpy().astype(np.int64)
    layer, vmax = adakv.Layer.from_workload(wl), float(Vc.float().abs().max())
    out, lse = adakv.decode_attn(layer, q[0], cu, hr, Kc, Vc, lens, want_lse=True)
    ref = D.decode_attention(to_f64(q[0]), oK, oV, cuh, hr, olen, g)
    _assert_decode_close(out, lse, *ref, vmax, "attention")
    full = torch.zeros(1, dtype=torch.int32, device=DEV)
    out, lse = adakv.decode_step(layer, q[0], kn[0], vn[0], cu, hr, Kc, Vc, lens, overflow=full, want_lse=True)
    D.append(oK, oV, cuh, hr, olen, to_f64(kn[0]).reshape(-1, d), to_f64(vn[0]).reshape(-1, d))
    assert int(full) == 1 and np.array_equal(lens.cpu().numpy(), olen)
    _assert_decode_close(out, lse, *D.decode_attention(to_f64(q[0]), oK, oV, cuh, hr, olen, g), vmax, "step")
    assert np.array_equal(to_f64(Kc), oK) and np.array_equal(to_f64(Vc), oV)
