"""A decoding step's checks in native code hand over exactly what the checks in Python hand over, and leave every call
that is not as it has to be to them (which then raise what they always raised)."""
import ctypes

import pytest
import torch

import paper_2407_11550_amd as adakv
from paper_2407_11550_amd import binding

H_Q, H_KV, D, BATCH, HEADROOM = 8, 2, 64, 2, 3
NSEG = BATCH * H_KV
P, I = ctypes.c_void_p, ctypes.c_int32
STEP = ctypes.CFUNCTYPE(ctypes.c_int, P, P, P, P, P, I, P, P, P, P, P, P, P, ctypes.c_size_t, P)


def arguments(device, dtype=torch.bfloat16):
    layer = adakv.Layer(dtype, H_Q, H_KV, D, 4, 3, 0.2, [50, 70], [40, 48])
    rows = sum(layer.B) + NSEG * HEADROOM
    g = torch.Generator().manual_seed(3)
    f = lambda *shape: torch.randn(*shape, generator=g).to(dtype).to(device)
    i = lambda *values: torch.tensor(values, dtype=torch.int32, device=device)
    cu = i(0, 20, 40, 64, 88)
    return layer, dict(q_new=f(BATCH, H_Q, D), k_new=f(BATCH, H_KV, D), v_new=f(BATCH, H_KV, D), cu_seqlens=cu,
                       headroom=HEADROOM, K_cache=f(rows, D), V_cache=f(rows, D), seg_len=i(20, 20, 24, 24),
                       overflow=i(0), out=torch.zeros(BATCH, H_Q, D, device=device), lse=torch.zeros(BATCH, H_Q, device=device),
                       ws=torch.zeros(adakv.decode_workspace_bytes(layer, HEADROOM), dtype=torch.uint8, device=device))


def native(layer, a, fn, stream=7):
    return binding._marshal.decode_step(ctypes.cast(fn, P).value, ctypes.addressof(layer.c), *a.values(), stream)


def strided(t):
    """The same values, every other element of a tensor twice as long."""
    return torch.stack([t, t], dim=-1)[..., 0]


# what each argument may be spoiled by; the native checks leave all of them to the ones in Python
SPOILED = {
    "q_shape": lambda a: a.update(q_new=a["q_new"][:, :-1].contiguous()),
    "q_order": lambda a: a.update(q_new=a["q_new"].transpose(1, 2).contiguous().transpose(1, 2)),
    "k_order": lambda a: a.update(k_new=a["k_new"].transpose(1, 2).contiguous().transpose(1, 2)),
    "v_shape": lambda a: a.update(v_new=a["v_new"][:1]),
    "q_type": lambda a: a.update(q_new=a["q_new"].to(torch.float16)),
    "cu_short": lambda a: a.update(cu_seqlens=a["cu_seqlens"][:NSEG]),
    "cu_type": lambda a: a.update(cu_seqlens=a["cu_seqlens"].long()),
    "headroom_too_large": lambda a: a.update(headroom=HEADROOM + 1),
    "cache_short": lambda a: a.update(K_cache=a["K_cache"][:-1]),
    "cache_order": lambda a: a.update(V_cache=a["V_cache"].t().contiguous().t()),
    "cache_width": lambda a: a.update(V_cache=a["V_cache"].view(-1, D // 2)),
    "cache_without_rows": lambda a: a.update(K_cache=a["K_cache"].new_empty(a["K_cache"].shape[0], 0, D)),
    "cu_strided": lambda a: a.update(cu_seqlens=strided(a["cu_seqlens"])),
    "len_strided": lambda a: a.update(seg_len=strided(a["seg_len"])),
    "out_strided": lambda a: a.update(out=strided(a["out"])),
    "lse_strided": lambda a: a.update(lse=strided(a["lse"])),
    "ws_strided": lambda a: a.update(ws=strided(a["ws"])),
    "len_short": lambda a: a.update(seg_len=a["seg_len"][:-1]),
    "overflow_empty": lambda a: a.update(overflow=a["overflow"][:0]),
    "out_short": lambda a: a.update(out=a["out"][:1]),
    "lse_short": lambda a: a.update(lse=a["lse"][:1]),
    "lse_type": lambda a: a.update(lse=a["lse"].double()),
    "ws_type": lambda a: a.update(ws=a["ws"].view(torch.int8)),
}


def test_tensors_of_the_host_and_others_are_not_taken(lib):
    assert binding._marshal is not None, "lib/_marshal.so is not built"
    layer, a = arguments("cpu")
    calls = []
    fn = STEP(lambda *given: calls.append(given) or 0)
    assert native(layer, a, fn) is None
    for other in (dict(q_new=None), dict(q_new=torch.nn.Parameter(a["q_new"])), dict(headroom=-1), dict(headroom=2.0),
                  dict(headroom=1 << 40), dict(ws=3)):
        assert native(layer, dict(a, **other), fn) is None
    assert native(layer, a, fn, stream=None) is None and not calls


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32])
@pytest.mark.parametrize("without", [(), ("overflow",), ("overflow", "lse")])
def test_what_is_handed_over(dtype, without):
    layer, a = arguments("cuda:0", dtype)
    a.update(dict.fromkeys(without))
    calls = []
    fn = STEP(lambda *given: calls.append(given) or 5)
    assert native(layer, a, fn) == 5
    address = {k: None if v is None else v if isinstance(v, int) else v.data_ptr() for k, v in a.items()}
    assert calls == [(ctypes.addressof(layer.c), *address.values(), a["ws"].numel(), 7)]


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(SPOILED))
def test_a_spoiled_argument_raises_as_without_the_native_checks(name, monkeypatch):
    layer, a = arguments("cuda:0")
    SPOILED[name](a)
    said = []
    for module in (binding._marshal, None):
        monkeypatch.setattr(binding, "_marshal", module)
        with pytest.raises((ValueError, adakv.AdaKVError)) as e:
            adakv.decode_step(layer, **a)
        said.append((type(e.value), str(e.value)))
    assert said[0] == said[1]


@pytest.mark.gpu
def test_a_refusal_of_the_library_and_the_results(lib, monkeypatch):
    got = []
    for module in (binding._marshal, None):
        monkeypatch.setattr(binding, "_marshal", module)
        layer, a = arguments("cuda:0")
        with pytest.raises(adakv.AdaKVError, match="adakv_decode_step"):
            adakv.decode_step(layer, **dict(a, ws=a["ws"][:0]))
        out, lse = adakv.decode_step(layer, **a)
        assert out is a["out"] and lse is a["lse"]
        assert adakv.decode_step(layer, **dict(a, lse=None)) is a["out"]
        got.append([a[k].cpu() for k in ("out", "lse", "K_cache", "V_cache", "seg_len", "overflow")])
    assert all(torch.equal(x, y) for x, y in zip(*got))


# h_q, h_kv, d, w: at most d rows with the head-room, so that a flat tensor of d elements has as many "rows" as are asked for
FLAT = adakv.Layer(torch.bfloat16, 2, 1, 128, 4, 3, 0.2, [50], [40])


@pytest.mark.parametrize("name", ["K_cache", "V_cache", "cu_seqlens", "seg_len", "out", "lse", "ws"])
def test_memory_the_kernels_would_miss_is_refused(name, lib):
    """A cache of one row of d elements, and buffers whose elements do not lie one behind the other: the checks in
    Python refuse them by name (here before they look at the device)."""
    f, i = (lambda *s: torch.zeros(*s, dtype=torch.bfloat16)), (lambda *v: torch.tensor(v, dtype=torch.int32))
    a = dict(K_cache=f(43, 128), V_cache=f(43, 128), cu_seqlens=i(0, 40), seg_len=i(40), out=torch.zeros(1, 2, 128),
             lse=torch.zeros(1, 2), ws=torch.zeros(adakv.decode_workspace_bytes(FLAT, 3), dtype=torch.uint8))
    if name == "seg_len":                       # (one segment's length is one element, strided or not)
        with pytest.raises(ValueError, match="must be a device tensor"):
            adakv.decode_attn(FLAT, f(1, 2, 128), headroom=3, **dict(a, seg_len=strided(a["seg_len"])))
        return
    a[name] = f(128) if "cache" in name else strided(a[name])
    with pytest.raises(ValueError, match=name):
        adakv.decode_attn(FLAT, f(1, 2, 128), headroom=3, **a)


@pytest.mark.gpu
def test_a_flat_cache_and_rows_further_on(lib):
    """The native checks leave a flat cache to the ones in Python; a buffer that is dense as far as it is used is taken."""
    calls = []
    fn = STEP(lambda *given: calls.append(given) or 0)
    f, i = (lambda *s: torch.zeros(*s, dtype=torch.bfloat16, device="cuda:0")), (lambda *v: torch.tensor(v, dtype=torch.int32, device="cuda:0"))
    a = dict(q_new=f(1, 2, 128), k_new=f(1, 1, 128), v_new=f(1, 1, 128), cu_seqlens=i(0, 40), headroom=3, K_cache=f(43, 128),
             V_cache=f(43, 128), seg_len=i(40), overflow=None, out=torch.zeros(1, 2, 128, device="cuda:0"), lse=None,
             ws=torch.zeros(adakv.decode_workspace_bytes(FLAT, 3), dtype=torch.uint8, device="cuda:0"))
    assert native(FLAT, a, fn) == 0 and len(calls) == 1
    for name in ("K_cache", "V_cache"):
        assert native(FLAT, dict(a, **{name: f(128)}), fn) is None
        with pytest.raises(ValueError, match=name):
            adakv.decode_step(FLAT, **dict(a, **{name: f(128)}))
    wide = torch.zeros(3, 4, 128, device="cuda:0")[:, :2]        # the first [2, 128] lie together
    assert adakv.decode_step(FLAT, **dict(a, out=wide)) is wide and len(calls) == 1


def test_host_tensors_are_named_where_there_is_no_gpu(lib):
    """... and not the missing GPU, which the stream is asked of."""
    layer, a = arguments("cpu")
    with pytest.raises(ValueError, match="q_new must be a device tensor"):
        adakv.decode_step(layer, **a)


@pytest.mark.parametrize("why", [RuntimeError("g++ failed on marshal.cpp"), FileNotFoundError("g++")])
def test_the_library_is_built_without_the_native_checks(why, monkeypatch, capsys, lib):
    import __graft_entry__ as entry
    from paper_2407_11550_amd import build

    def fails():
        raise why
    monkeypatch.setattr(build, "build", lambda: adakv.library_path())
    monkeypatch.setattr(build, "build_marshal", fails)
    monkeypatch.setattr(build, "build_abi_driver", lambda: "driver")
    entry.build()
    said = capsys.readouterr().out
    assert "built " + adakv.library_path() in said and f"not built: a decoding step's native checks, the ones in Python do the same ({why})" in said
