"""The extension module that makes the calls with plain tensors writes the descriptors and options that the ctypes binding
writes, and leaves alone what it does not take.  No device: a Python callback stands in for the library's entry point."""
import ctypes

import pytest
import torch

from paper_2508_08192_amd import treeattn as ta

P = ctypes.POINTER(ta.ta_tensor)


@pytest.fixture()
def captured(monkeypatch):
    ta.load_library()
    seen = []

    def entry(n, opts):
        def fn(*args):
            plain = args[:n + 1] if opts else args
            seen.append(([(bytes(a.contents) if a else None) if isinstance(a, P) else a for a in plain],))
            if opts:
                o = ta.ta_opts.from_buffer_copy(args[n + 1].contents)
                seen[-1] += ([bytes(x.contents) if x else None for x in (o.k_new, o.v_new)],)
                o.k_new = o.v_new = None
                seen[-1] += (bytes(o),)
            return 7
        return fn

    T8, V = [P] * 8, ctypes.c_void_p
    cbs = {"tree_attn_fwd": ctypes.CFUNCTYPE(ctypes.c_int, *T8, V)(entry(8, False)),
           "tree_attn_fwd_ex": ctypes.CFUNCTYPE(ctypes.c_int, *T8, V, ctypes.POINTER(ta.ta_opts))(entry(8, True)),
           "tree_attn_append": ctypes.CFUNCTYPE(ctypes.c_int, *[P] * 6, V)(entry(6, False)),
           "tree_attn_compact": ctypes.CFUNCTYPE(ctypes.c_int, *[P] * 6, ctypes.c_int32, P, V)(entry(6, False))}
    cbs["tree_attn_fwd_static"] = cbs["tree_attn_fwd_ex"]

    class Lib:
        pass
    lib = Lib()
    lib.tree_attn_strerror = lambda status: b"the entry says so"
    for name, cb in cbs.items():
        setattr(lib, name, cb)
        monkeypatch.setitem(ta._entry, name, ctypes.cast(cb, ctypes.c_void_p).value)
    monkeypatch.setattr(ta, "_lib", lib)
    return seen


def _tensors():
    q = torch.zeros(2, 3, 4, 8, dtype=torch.bfloat16)
    k = torch.zeros(5, 2, 16, 9, dtype=torch.bfloat16)[..., 1:]
    return [q, k, k.transpose(1, 2), torch.zeros(2, 4, dtype=torch.int32)[:, :2], torch.zeros(2, dtype=torch.int32),
            torch.zeros(3, dtype=torch.int32), torch.empty(0, 3, 4, 8), torch.zeros(2, 4, 3, dtype=torch.float64)]


class Sub(torch.Tensor):
    pass


def _both(call, seen, monkeypatch):
    """The call through the module and through ctypes: (module result, ctypes result, was the module's answer used)."""
    used = []
    real = ta._call

    class Spy:
        def __getattr__(self, name):
            def f(*a):
                used.append(getattr(real, name)(*a))
                return used[-1]
            return f
    res = []
    for mod in (Spy(), None):
        monkeypatch.setattr(ta, "_call", mod)
        try:
            res.append(call())
        except Exception as e:
            res.append(type(e))
        res.append(seen.pop() if seen else None)
    monkeypatch.setattr(ta, "_call", real)

    assert res[0] == res[2] and res[1] == res[3]
    return res[0], bool(used) and used[-1] is not None


def test_plain_tensors_are_described_as_through_ctypes(captured, monkeypatch):
    t = _tensors()
    par = torch.nn.Parameter(t[0], requires_grad=False)
    odd = [torch.zeros((), dtype=torch.int32), torch.zeros(1, 1, 1, 1, 1), torch.zeros(3, 1).expand(3, 7), par]
    for args in (t, t[:3] + [None] + t[4:7] + [None], odd + odd):
        assert _both(lambda: ta.tree_attn_fwd(*args, stream=0x1234, check=False), captured, monkeypatch) == (7, True)
        assert _both(lambda: ta.tree_attn_append(*args[:6], stream=0, check=False), captured, monkeypatch) == (7, True)
        assert _both(lambda: ta.tree_attn_compact(*args[:6], 9, seq_lens_out=args[7], stream=0, check=False), captured,
                     monkeypatch) == (7, True)


@pytest.mark.parametrize("kw", [
    {}, {"scale": 0.25, "num_splits": 3, "kernel": 2, "item_cost": 4096, "q_node_offset": 5},
    {"tree_masks": torch.zeros(2, 3, dtype=torch.int64)[:, :2], "kv_start": torch.zeros(2, dtype=torch.int32)},
    {"tree_masks": torch.zeros(3, dtype=torch.int64), "k_new": torch.zeros(2, 3, 2, 8), "v_new": torch.zeros(2, 3, 2, 8)[:1]},
    {"scale": float("nan")}, {"num_splits": -1}])
def test_options_are_those_of_ctypes(captured, monkeypatch, kw):
    t = _tensors()
    for fn in (ta.tree_attn_fwd_ex, ta.tree_attn_fwd_static):
        assert _both(lambda: fn(*t, stream=0, check=False, **kw), captured, monkeypatch) == (7, True)


def test_what_is_not_of_the_simple_form_goes_through_ctypes(captured, monkeypatch):
    t = _tensors()
    d = ta.Desc((2, 3, 4, 8), ta.TA_BF16)
    for args in ([d] + t[1:], [t[0].as_subclass(Sub)] + t[1:]):
        assert _both(lambda: ta.tree_attn_fwd(*args, stream=0, check=False), captured, monkeypatch) == (7, False)
    for kw in ({"scale": 1}, {"num_splits": True}, {"status": torch.zeros(1, dtype=torch.int32)},
               {"workspace": torch.zeros(8)}, {"k_new": d, "v_new": d}):
        assert _both(lambda: ta.tree_attn_fwd_ex(*t, stream=0, check=False, **kw), captured, monkeypatch) == (7, False)
    # errors are the binding's own: six dimensions, a number for a tensor, an option that is none, a meta tensor's address
    assert _both(lambda: ta.tree_attn_fwd(torch.zeros([1] * 6), *t[1:], stream=0), captured, monkeypatch)[0] is ValueError
    assert _both(lambda: ta.tree_attn_fwd(3, *t[1:], stream=0), captured, monkeypatch)[0] is AttributeError
    assert _both(lambda: ta.tree_attn_fwd_ex(*t, stream=0, num_splits="x"), captured, monkeypatch)[0] is ValueError
    with pytest.raises(ta.TreeAttnError):
        ta.tree_attn_fwd(*t, stream=0)


def test_the_library_works_without_the_module():
    """Where the extension module cannot be imported the binding warns and calls through ctypes.  In a process of its own."""
    import os
    import subprocess
    import sys
    code = ("import sys, warnings\n"
            "sys.modules['paper_2508_08192_amd._call'] = None\n"
            "import torch\n"
            "from paper_2508_08192_amd import treeattn as ta\n"
            "with warnings.catch_warnings(record=True) as seen:\n"
            "    warnings.simplefilter('always')\n"
            "    assert ta.tree_attn_version() > 0\n"
            "assert ta._call is None and any('ctypes' in str(w.message) for w in seen)\n"
            "q = torch.zeros(2, 3, 4, 64)\n"
            "assert ta.tree_attn_fwd(q, q, None, None, q, q, q, stream=0, check=False) == ta.TA_ERR_NULL\n"
            "assert ta.tree_attn_append(q, q, q, q, None, q, stream=0, check=False) == ta.TA_ERR_DTYPE\n"
            "print('ok')\n")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = subprocess.run([sys.executable, "-c", code], cwd=root, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert out.returncode == 0 and "ok" in out.stdout, out.stdout


def test_a_build_without_a_host_compiler_leaves_the_library(monkeypatch, tmp_path):
    from paper_2508_08192_amd import build
    monkeypatch.setattr(build, "LIB", str(tmp_path / "lib.so"))
    monkeypatch.setattr(build, "CALL_MODULE", str(tmp_path / "_call.so"))
    monkeypatch.setattr(build, "generate_blocks", lambda verbose: None)
    monkeypatch.setattr(build, "verify_register_partition", lambda verbose: None)
    hipcc = tmp_path / "hipcc"
    hipcc.write_text('#!/bin/sh\nwhile [ $# -gt 1 ]; do [ "$1" = -o ] && : > "$2"; shift; done\n')
    hipcc.chmod(0o755)
    monkeypatch.setenv("HIPCC", str(hipcc))
    monkeypatch.setenv("CXX", str(tmp_path / "no_such_compiler"))
    (tmp_path / "_call.so").write_text("of other sources")
    assert build.build_library() == str(tmp_path / "lib.so") and (tmp_path / "lib.so").exists()
    assert not (tmp_path / "_call.so").exists()


def test_any_zero_is_the_default_stream(captured, monkeypatch):
    import numpy as np
    t = _tensors()
    for zero in (0, 0.0, np.int64(0), False):
        assert _both(lambda: ta.tree_attn_fwd(*t, stream=zero, check=False), captured, monkeypatch)[0] == 7
        assert _both(lambda: ta.tree_attn_fwd_ex(*t, stream=zero, check=False), captured, monkeypatch)[0] == 7
    assert _both(lambda: ta.tree_attn_fwd(*t, stream="x", check=False), captured, monkeypatch)[0] is AttributeError
