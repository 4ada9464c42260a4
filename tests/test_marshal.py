"""The native argument checks in front of the calls that are made step after step: the same results, bit for bit, and the same
refusals as the Python beside them, which every call that is not plain still goes through."""
import os
import subprocess
import sys

import pytest
import torch

from paper_2404_09526_amd import workloads as wl


ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


class Plainless(torch.Tensor):
    """A subclass: not plain, so its calls take the Python route."""


def calls(esp, cuda):
    """name -> (function, keyword arguments with everything given, names of its outputs)"""
    pc = wl.contiguous_prefill("marshal", 40, 60, [(0, 50), (50, 100)], 8, 2, 71, cuda)
    dc = wl.decode_pool("marshal", [5, 0, 300], 1024, 8, 2, 72, cuda, n_new=0, n_peers=2)
    ws = torch.empty(1 << 20, dtype=torch.uint8, device=cuda)
    out = lambda n, dt=torch.bfloat16: dict(O=torch.zeros((n, 8, 128), dtype=dt, device=cuda), LSE=torch.zeros((n, 8), device=cuda))
    s = pc.shards[0]
    pre = dict(q=pc.q, k=s.k, v=s.v, q_pos=pc.q_pos, kv_pos=s.kv_pos, softmax_scale=pc.scale, workspace=ws)
    two = lambda n: torch.tensor([0, 7, n], dtype=torch.int32, device=cuda)
    dec = dict(q=dc.q, k_pool=dc.k_pool, v_pool=dc.v_pool, slot_idx=dc.slot_idx, seq_offsets=dc.seq_offsets, max_len=300, softmax_scale=None, workspace=ws)
    parts = [out(3, torch.float32) for _ in range(2)]
    new = torch.randn((3, 2, 128), device=cuda).bfloat16()
    return {
        "prefill": (esp.esp_partial_attn_prefill, pre | out(40), ("O", "LSE")),
        "prefill-batch-f32": (esp.esp_partial_attn_prefill, pre | out(40, torch.float32) | dict(cu_q=two(40), cu_kv=two(50), max_q=33, max_kv=43, causal=False), ("O", "LSE")),
        "decode": (esp.esp_partial_attn_decode, dec | out(3), ("O", "LSE")),
        "decode-merge": (esp.esp_partial_attn_decode_merge, dec | out(3) | dict(peer_O=list(dc.peer_O), peer_LSE=tuple(dc.peer_LSE)), ("O", "LSE")),
        "merge-f32": (esp.esp_merge_partials, dict(O_parts=[p["O"].normal_() for p in parts], LSE_parts=[p["LSE"].normal_() for p in parts]) | out(3), ("O", "LSE")),
        "append": (esp.esp_kv_append, dict(k=new, v=-new, slot_idx=torch.tensor([4, -1, 9], dtype=torch.int32, device=cuda),
                                           k_pool=torch.zeros((16, 2, 128), dtype=torch.bfloat16, device=cuda),
                                           v_pool=torch.zeros((16, 2, 128), dtype=torch.bfloat16, device=cuda)), ("k_pool", "v_pool")),
    }


NAMES = ["prefill", "prefill-batch-f32", "decode", "decode-merge", "merge-f32", "append"]


@pytest.mark.gpu
@pytest.mark.parametrize("name", NAMES)
def test_native_checks_make_the_same_call(cuda, monkeypatch, name):
    from paper_2404_09526_amd import binding as esp
    call, kw, outs = calls(esp, cuda)[name]
    taken = []

    class Spy:
        def __getattr__(self, what):
            f = getattr(marshal, what)
            return lambda *a: (taken.append(f(*a)), taken[-1])[1]
    marshal = esp._marshal
    monkeypatch.setattr(esp, "_marshal", Spy())
    results = []
    for plain in (True, False):
        first = next(iter(kw))
        t = kw[first]
        odd = [t[0].as_subclass(Plainless)] + list(t[1:]) if isinstance(t, list) else t.as_subclass(Plainless)
        for o in outs:
            kw[o].zero_()
        call(**(kw if plain else kw | {first: odd}))
        torch.cuda.synchronize()
        results.append([kw[o].clone() for o in outs])
    assert taken == [0, None]
    for a, b in zip(*results):
        assert a.any() and torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.gpu
@pytest.mark.parametrize("name", NAMES)
def test_what_was_refused_stays_refused(cuda, name):
    """One tensor at a time on the host, of another type, or not contiguous; a workspace that is too small; sizes that do not match."""
    from paper_2404_09526_amd import binding as esp
    call, kw, _ = calls(esp, cuda)[name]
    for key, t in kw.items():
        if not isinstance(t, torch.Tensor) or key == "workspace":
            continue
        wide = torch.stack([t, t], dim=-1)[..., 0]
        for bad in (t.cpu(), t.to(torch.float64), wide):
            with pytest.raises(ValueError):
                call(**(kw | {key: bad}))
    if "workspace" in kw:
        with pytest.raises(esp.EspError) as e:
            call(**(kw | {"workspace": kw["workspace"][:128]}))
        assert e.value.status == esp.ESP_ERR_WORKSPACE
    shorter = {"prefill": "q_pos", "prefill-batch-f32": "cu_kv", "decode": "seq_offsets", "decode-merge": "seq_offsets", "append": "slot_idx"}
    if name in shorter:
        with pytest.raises(ValueError):
            call(**(kw | {shorter[name]: kw[shorter[name]][:-1].contiguous()}))


@pytest.mark.gpu
@pytest.mark.parametrize("name", NAMES[:-1])
def test_an_output_too_small_for_what_is_written_is_refused(cuda, name):
    """One row short, of another type, on the host or spread out; a larger output is the caller's business and is written as far as
    the call goes.  A workspace on the host, or one whose bytes are not its own."""
    from paper_2404_09526_amd import binding as esp
    call, kw, outs = calls(esp, cuda)[name]
    names = [name] + (["decode-static"] if name == "decode" else [])
    for which in names:
        if which == "decode-static":
            call, kw = esp.esp_partial_attn_decode_static, {k: v for k, v in kw.items() if k != "workspace"}
        for key in outs:
            t = kw[key]
            for bad in (t[:-1].contiguous(), t.to(torch.float16), t.cpu(), torch.stack([t, t], dim=-1)[..., 0]):
                with pytest.raises(ValueError):
                    call(**(kw | {key: bad}))
        if not name.startswith("prefill"):                          # (prefill asks for the very shape)
            for o in outs:
                kw[o].zero_()
            call(**kw)
            room = {o: torch.full((kw[o].shape[0] + 2,) + kw[o].shape[1:], 7, dtype=kw[o].dtype, device=cuda) for o in outs}
            call(**(kw | room))
            torch.cuda.synchronize()
            for o in outs:
                n = kw[o].shape[0]
                assert torch.equal(room[o][:n], kw[o]) and (room[o][n:] == 7).all()
        if "workspace" in kw:
            for bad in (kw["workspace"].cpu(), kw["workspace"][:1].expand(1 << 20), kw["workspace"][::2]):
                with pytest.raises(ValueError):
                    call(**(kw | {"workspace": bad}))


def test_the_native_checks_are_loaded_for_this_torch_only_and_can_be_missing(monkeypatch):
    """Built for another torch, or not built, they are not looked at: the package comes up on its Python checks, and a build is due."""
    code = ("from paper_2404_09526_amd import build; build.marshal_path = lambda: '/nonexistent/_marshal.so'\n"
            "from paper_2404_09526_amd import binding as b\n"
            "assert b._marshal.decode(1, 2) is None and b._marshal.merge() is None and 'gfx950' in b.version()")
    subprocess.run([sys.executable, "-c", code], check=True, cwd=ROOT)
    from paper_2404_09526_amd import binding, build
    build.build_lib(force=False)
    assert not build.is_stale() and binding._load_marshal() is not binding._PythonAlone
    here = build.marshal_path()
    monkeypatch.setattr(torch, "__version__", "0.0.1+other")
    assert build.marshal_path() != here and build.is_stale() and binding._load_marshal() is binding._PythonAlone
