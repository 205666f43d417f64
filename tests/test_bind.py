"""The per-token calls marshalled in C (csrc/rk_bind.cpp) hand the library the arguments that the ctypes path hands it, or leave the call to
that path: both are pointed at entry points that write down what arrives."""
import ctypes as C
import os
import subprocess
import sys
import types

import numpy as np
import pytest
import torch

import paper_2605_19218_amd as rk

B, HQ, HKV, CAP = 2, 8, 2, 64
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
vp, f32, sz, i32 = C.c_void_p, C.c_float, C.c_size_t, C.c_int
PL, PT = C.POINTER(rk.rk_layout), C.POINTER(rk.rk_text)
SIGNATURES = {
    "rk_decode_attn": [vp, PL, vp, vp, vp, vp, vp, f32, vp, vp, sz, vp],
    "rk_append_decode_attn": [vp, PL, vp, vp, vp, vp, vp, vp, vp, vp, f32, vp, vp, sz, vp],
    "rk_decode_attn_dual": [vp, PL, vp, vp, vp, vp, vp, PT, f32, vp, vp, sz, vp],
    "rk_append_text_decode_attn_dual": [vp, PL, vp, vp, vp, vp, vp, vp, vp, PT, f32, vp, vp, sz, vp],
}


class Duck:
    """anything with data_ptr()"""

    def data_ptr(self):
        return 4096

    def numel(self):
        return 10

    def element_size(self):
        return 3


class OtherLayout(rk.Layout):
    def c(self):
        x = super().c()
        x.keep = 5
        return x


def tensor(*shape):
    return torch.zeros(*shape, dtype=torch.bfloat16)


def layout(cls=rk.Layout, **more):
    return cls(B, HQ, HKV, 16, rk.RK_BF16, CAP, 40, **{"seq_len": torch.zeros(B, dtype=torch.int32), **more})


def text(**more):
    k = tensor(B, HKV, 48, 128)
    return rk.Text(k, tensor(B, HKV, 48, 128), 33, **{"len": torch.zeros(B, dtype=torch.int32), **more})


@pytest.fixture
def paths(monkeypatch):
    """record(name, positional, keywords, fast): the arguments that reached the entry point"""
    rk.lib()
    if rk._bind is None:
        pytest.fail("_rkbind.so is not built")
    seen, keep = [], []

    def entry(kinds):
        def f(*a):
            row = []
            for x, kind in zip(a, kinds):
                if kind in (PL, PT):
                    row.append([getattr(x.contents, n) for n, _ in x.contents._fields_] if x else None)
                else:
                    row.append(x)
            seen.append(row)
            return 0
        return C.CFUNCTYPE(i32, *kinds)(f)

    stub = types.SimpleNamespace()
    for name, kinds in SIGNATURES.items():
        keep.append(entry(kinds))
        f = keep[-1]
        f.argtypes, f.restype = kinds, i32
        setattr(stub, name, f)
    real, bind = rk.lib(), rk._bind
    bind.bind(rk.Layout, rk.Text, *[C.cast(getattr(stub, n), vp).value for n in SIGNATURES])

    def record(name, args, kw, fast):
        seen.clear()
        monkeypatch.setattr(rk, "_bind", bind if fast else None)
        monkeypatch.setattr(rk, "_lib", None if fast else stub)
        if fast:                                    # the ctypes path must not be needed
            monkeypatch.setattr(rk, "lib", lambda: pytest.fail("the ctypes path was taken"))
        getattr(rk, name)(*args, **kw)
        monkeypatch.undo()
        assert len(seen) == 1
        return list(seen[0])

    yield record, bind
    bind.bind(rk.Layout, rk.Text, *[C.cast(getattr(real, n), vp).value for n in SIGNATURES])


def call(name, lay, txt, ws, scale=0.0, kv=None, ctx=77):
    """positional arguments of an entry point; kv: in the place of a tensor"""
    t = [tensor(4, 16) for _ in range(8)]
    if kv is not None:
        t[1] = kv
    out = tensor(4, 16)
    if name == "rk_decode_attn":
        return [ctx, lay, *t[:5], scale, out, ws]
    if name == "rk_append_decode_attn":
        return [ctx, lay, *t[:8], scale, out, ws]
    if name == "rk_decode_attn_dual":
        return [ctx, lay, *t[:5], txt, scale, out, ws]
    return [ctx, lay, *t[:7], txt, scale, out, ws]


@pytest.mark.parametrize("name", list(SIGNATURES))
def test_same_arguments(paths, name):
    record, _ = paths
    ws = torch.empty(1000, dtype=torch.float32)
    forms = [
        (call(name, layout(), text(), ws), {}),
        (call(name, layout(seq_len=None, head_dim=64), text(len=None), ws, scale=0.25), {"stream": 12345}),
        (call(name, layout(seq_len=1 << 47), text(strides=(9, 8, 7), capacity=40), None, scale=1), {"stream": None}),
        (call(name, layout(), text(capacity=7), 1 << 40, kv=Duck()), {"workspace_bytes": 99}),
        (call(name, layout(), text(), Duck(), kv=None, ctx=None), {"stream": types.SimpleNamespace(cuda_stream=321)}),
        (call(name, layout(), text(), ws, kv=(1 << 64) - 16), {"workspace_bytes": 0}),
    ]
    for args, kw in forms:
        assert record(name, args, kw, True) == record(name, args, kw, False)
    args = call(name, layout(), text(), ws)
    args[5] = None                                      # a missing tensor
    assert record(name, args, {}, True) == record(name, args, {}, False)


@pytest.mark.parametrize("name", list(SIGNATURES))
def test_other_forms_go_to_ctypes(paths, name):
    _, bind = paths
    fast = {"rk_decode_attn": bind.decode, "rk_append_decode_attn": bind.append_decode, "rk_decode_attn_dual": bind.dual,
            "rk_append_text_decode_attn_dual": bind.append_dual}[name]
    ws = torch.empty(10)
    odd = [call(name, layout(OtherLayout), text(), ws), call(name, layout(), text(), ws, scale="0.5"),
           call(name, layout(), text(), ws, kv=np.int64(4096)), call(name, layout(), text(), ws, kv=-16), call(name, layout(), text(), ws, kv="x"),
           call(name, layout(), text(), 4096), call(name, None, text(), ws), call(name, layout(), text(), ws, kv=True)]
    big = layout()
    big.capacity = 1 << 33
    odd.append(call(name, big, text(), ws))
    if "dual" in name:
        odd += [call(name, layout(), None, ws), call(name, layout(), text(strides=[1, 2, 3]), ws), call(name, layout(), text(strides=(1, 2)), ws)]
    for args in odd:
        assert fast(*args, None, None) is None


class Interrupted:
    def __init__(self):
        self.asked = 0

    def data_ptr(self):
        self.asked += 1
        if self.asked == 1:
            raise KeyboardInterrupt
        return 4096


@pytest.mark.parametrize("name", list(SIGNATURES))
def test_an_interrupt_is_not_swallowed(paths, name):
    """What comes once, out of an argument's own code, ends the call as it does on the ctypes path."""
    record, _ = paths
    with pytest.raises(KeyboardInterrupt):
        record(name, call(name, layout(), text(), torch.empty(10), kv=Interrupted()), {}, True)


def test_statuses():
    """Errors come out as from the ctypes path, with the library's text."""
    ctx = rk.rk_create(rk.RK_DEVICE_NONE)
    try:
        lay = layout()
        ws = torch.empty(rk.rk_decode_workspace_size(ctx, lay), dtype=torch.uint8)
        for change, status in (({}, rk.RK_ERR_NO_DEVICE), ({"keep": 0}, rk.RK_ERR_INVALID_ARG), ({"head_dim": 64}, rk.RK_ERR_UNSUPPORTED)):
            for k, v in change.items():
                setattr(lay, k, v)
            texts = []
            for bind in (rk._bind, None):
                old, rk._bind = rk._bind, bind
                try:
                    with pytest.raises(rk.RotateKError) as e:
                        rk.rk_decode_attn(*call("rk_decode_attn", lay, None, ws, ctx=ctx))
                finally:
                    rk._bind = old
                assert e.value.status == status
                texts.append(str(e.value))
            assert texts[0] == texts[1]
    finally:
        rk.rk_destroy(ctx)


def python(code, **env):
    res = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300, cwd=ROOT, env={**os.environ, **env})
    assert res.returncode == 0, res.stderr
    return res.stdout, res.stderr


def test_without_the_extension():
    """Where it cannot be imported the calls work through ctypes, and the first use says so."""
    out, err = python("import sys; sys.modules['paper_2605_19218_amd._rkbind'] = None\n"
                      "import paper_2605_19218_amd as rk\n"
                      "c = rk.rk_create(rk.RK_DEVICE_NONE); assert rk._bind is None\n"
                      "lay = rk.Layout(1, 4, 4, 16, rk.RK_BF16, 64, 40, seq_len=4096)\n"
                      "try: rk.rk_decode_attn(c, lay, 4096, 4096, 4096, 4096, 4096, 0.0, 4096, 4096, workspace_bytes=1 << 30)\n"
                      "except rk.RotateKError as e: print(e.status)")
    assert out.strip() == str(rk.RK_ERR_NO_DEVICE) and "RuntimeWarning" in err and "ctypes" in err


def test_build_without_a_host_compiler(tmp_path):
    """A missing compiler costs the extension, not the build; nothing of an earlier build is left to be loaded, and the file's name is
    for this interpreter alone."""
    stale = tmp_path / "_rkbind.so"
    stale.write_bytes(b"x")
    out, _ = python("from paper_2605_19218_amd import build\nimport os, sys\n"
                    "name = os.path.basename(build.BIND)\n"
                    f"build.HERE, build.BIND = {str(tmp_path)!r}, os.path.join({str(tmp_path)!r}, name)\n"
                    "print(build.build_bind(), os.listdir(build.HERE))\n"
                    "os.environ.pop('CXX')\n"
                    "print(build.build_bind() == build.BIND, os.listdir(build.HERE) == [name], name.split('.', 1)[1] != 'so')",
                    CXX=str(tmp_path / "no-such-compiler"))
    assert "WARNING" in out and "None []" in out and "True True True" in out
