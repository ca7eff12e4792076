"""The extension that marshals the frequent calls: for ordinary arguments it makes the same call as the Python code does, and
it leaves everything else to that code."""
import os
import sys
import sysconfig
import timeit

import pytest
import torch

from paper_2601_20499_amd import build
from tests import gpu_util as gu


@pytest.fixture(scope="module")
def b():
    from paper_2601_20499_amd import binding
    return binding


def test_what_is_not_ordinary_is_left_to_python(b):
    native = b._marshal()
    assert native and native is b._native
    q, ws = torch.zeros(2, 1, 64, dtype=torch.bfloat16), torch.zeros(1, dtype=torch.uint8)       # not on a GPU
    assert native.attn(q, q, q, q, q, [0, 0], [0], q, 0.125, None, None, ws, None, None, False) is None
    assert native.score(q, q, q, [0, 0], [0], ws, 0.125, 4, 0, ws, None, None) is None
    cache = b.Cache(None, None, [0, 10], [2], [8], d=64)
    assert native.append(cache, q, q, None) is None and native.pack(cache, [2], [8], q, q, None) is None
    assert native.attn(q) is None and native.append() is None
    with pytest.raises(TypeError):
        native.setup(1)


def test_what_is_left_to_python_is_left_quickly(b):
    """A call that is marshalled in Python all the same takes little more than before there was an extension: looking at its arguments costs less
    than twice what Python takes for one of its lists (a third here; six times with exceptions)."""
    native = b._marshal()
    q, ws, off, lens = torch.zeros(2, 12, 64, dtype=torch.bfloat16), torch.zeros(1, dtype=torch.uint8), [0] * 13, [0] * 12
    cache = b.Cache(None, None, off, lens, lens, d=64)
    looks = [lambda: native.attn(q, q, q, q, q, off, lens, q, 0.125, None, None, ws, None, None, False),
             lambda: native.score(q, q, q, off, lens, ws, 0.125, 4, 0, ws, None, None),
             lambda: native.append(cache, q, q, None), lambda: native.pack(cache, lens, lens, q, q, None)]
    best = lambda f: min(timeit.repeat(f, number=200, repeat=20))
    one_list = best(lambda: b._i32(lens))
    for look in looks:
        assert look() is None and best(look) < 2 * one_list


def test_the_extension_is_this_interpreters(b):
    assert b._marshal().__file__ == build.MARSHAL and build.MARSHAL.endswith(sysconfig.get_config_var("EXT_SUFFIX"))


@pytest.mark.parametrize("lacking", ["torch", "g++", "headers", "nothing"])
def test_the_library_is_built_where_the_extension_cannot_be(monkeypatch, tmp_path, capsys, lacking):
    """Only hipcc is needed for the library; what is missing for the extension is told, and none of an earlier build stays."""
    commands = []
    monkeypatch.setattr(build.subprocess, "run", lambda cmd, **_: commands.append(cmd[0]))
    monkeypatch.setattr(build, "PKG", str(tmp_path))
    monkeypatch.setattr(build, "MARSHAL", str(tmp_path / "_marshal.x.so"))
    for old in ("_marshal.x.so", "_marshal.so"):
        (tmp_path / old).write_text("")
    if lacking == "torch":
        monkeypatch.setitem(sys.modules, "torch", None)
    elif lacking == "g++":
        monkeypatch.setattr(build.shutil, "which", lambda _: None)
    elif lacking == "headers":
        monkeypatch.setattr(build, "marshal_includes", lambda _: [str(tmp_path)])
    assert build.build_library(verbose=False) == build.LIB
    assert [os.path.basename(c) for c in commands] == ["hipcc"] + ["g++"] * (lacking == "nothing")
    assert os.listdir(tmp_path) == []
    told = capsys.readouterr().out
    assert (told == "") == (lacking == "nothing") and (lacking in ("nothing", "headers") or lacking in told)


def test_lists_shorter_than_the_heads_are_refused(b):
    """The library reads a number per head (hist_off and head_row_off one more); no call reads past the end of a list."""
    q, ws = torch.zeros(2, 3, 64, dtype=torch.bfloat16), torch.zeros(1, dtype=torch.uint8)
    off, heads, short = [0] * 4, [0] * 3, [0] * 2
    cache = b.Cache(None, None, off, heads, heads, d=64)
    calls = [lambda **k: b.df_attn_fwd(q, q, q, q, q, k.get("off", off), k.get("sink", heads), q, 0.125, workspace=ws, hist_len=k.get("len")),
             lambda **k: b.df_attn_fwd_static(q, q, q, q, q, k.get("off", off), k.get("sink", heads), q, 0.125, hist_len=k.get("len")),
             lambda **k: b.df_head_score(q, q, q, k.get("off", off), k.get("sink", heads), ws, 0.125, workspace=ws, hist_len=k.get("len"))]
    for call in calls:
        for wrong in (dict(off=heads), dict(off=tuple(heads)), dict(sink=short), dict(len=short)):
            with pytest.raises(ValueError):
                call(**wrong)
    for wrong in ((short, heads), (heads, short)):
        for pack in (b.df_pack_context, b.prepared_pack):
            with pytest.raises(ValueError):
                pack(cache, *wrong, q, q)
    for wrong in ((heads, heads, heads), (off, heads, short)):
        with pytest.raises(ValueError):
            b.Cache(None, None, *wrong, d=64)
    with pytest.raises(ValueError):
        b.df_attn_plan(1, 1, heads, short)
    with pytest.raises(ValueError):
        b.df_attn_units(64, False, 1, 1, heads, short)


@pytest.mark.gpu
@pytest.mark.parametrize("d", [64, 128])
def test_native_and_python_marshalling_make_the_same_calls(b, monkeypatch, d):
    dev, H, T, Nq = gu.dev(), 3, 70, 140
    g = torch.Generator(device=dev).manual_seed(d)
    rnd = lambda *s: torch.randn(*s, generator=g, device=dev).to(torch.bfloat16)
    q, kc, vc = rnd(H, Nq, d).transpose(0, 1), rnd(Nq, H, d), rnd(Nq, H, d)
    sink, win = [T, 0, T], [2 * T, T, 0]
    off = [0, 3 * T, 4 * T, 5 * T]
    k0, v0 = rnd(5 * T, d), rnd(5 * T, d)
    ws = torch.empty(b.df_attn_workspace_bytes(H, d, Nq), dtype=torch.uint8, device=dev)

    def results():
        out = [torch.zeros(Nq, H, d, dtype=torch.bfloat16, device=dev) for _ in range(4)]
        F, F2, lse = torch.zeros(H, 3, device=dev), torch.zeros(H, 3, device=dev), torch.zeros(H, Nq, device=dev)
        scale = d ** -0.5
        b.df_attn_fwd(q, kc, vc, k0, v0, off, sink, out[0], scale, lse_out=lse, score_out=F, workspace=ws)
        b.df_attn_fwd(q, kc, vc, k0, v0, tuple(off), None, out[1], scale, workspace=ws, hist_len=[T, T, 5], stream=0)
        b.df_attn_fwd_static(q, kc, vc, k0, v0, off, sink, out[2], scale, stream=torch.cuda.current_stream())
        b.df_attn_fwd(q, kc, vc, None, None, [0] * (H + 1), [0] * H, out[3], scale, workspace=ws)
        b.df_head_score(q, kc, k0, off, sink, F2, scale, q_sample_stride=3, q_offset=1, workspace=ws, hist_len=[3 * T, T, T])
        cache = b.Cache(k0.clone(), v0.clone(), off, sink, win, d)
        for _ in range(2):
            b.df_kv_append(cache, kc, vc)
        kp, vp = torch.zeros_like(k0), torch.zeros_like(v0)
        packed = b.df_pack_context(cache, sink, win, kp, vp)
        assert type(packed) is tuple and all(type(x) is list for x in packed)
        errors = []
        for call in (lambda: b.df_attn_fwd(q, kc, vc, k0, v0, off, [T + 1, T + 1, 0], out[0], scale, workspace=ws),
                     lambda: b.df_attn_fwd(q, kc, vc, k0, v0, off, sink, out[0], scale),
                     lambda: b.df_attn_fwd(q, kc, vc[:, :, :], k0, v0, off, sink, out[0], -1.0, workspace=ws),
                     lambda: b.df_head_score(q, kc, k0, off, sink, F2, scale, q_sample_stride=0, workspace=ws),
                     lambda: b.df_pack_context(cache, sink, win, kp[:5], vp)):
            with pytest.raises(b.DfError) as e:
                call()
            errors.append((e.value.status, str(e.value)))
        for call in (lambda: b.df_attn_fwd(q, kc, q, k0, v0, off, sink, out[0], scale, workspace=ws),
                     lambda: b.df_kv_append(cache, kc, q)):
            with pytest.raises(AssertionError):      # strides of keys and values that differ
                call()
        torch.cuda.synchronize()
        return [*out, F, F2, lse, cache.k_cache, cache.v_cache, kp, vp], [packed, cache.win_len[:], cache.win_pos[:], cache.sink_len[:], errors]

    native = b._marshal()
    assert native
    monkeypatch.setattr(b, "_native", native)
    tensors, numbers = results()
    monkeypatch.setattr(b, "_native", False)
    for x, y in zip(tensors, results()[0]):
        assert torch.equal(x, y) and x.float().abs().sum() > 0
    assert numbers == results()[1]
