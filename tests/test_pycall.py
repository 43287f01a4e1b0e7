"""The native calls of the per-step functions give what ctypes gives: the same
status and message for the same arguments (no GPU: every call here is refused
or is a no-op), for pointers as None, integers and tensors, and for integers
that are not Python ints; wrong counts and types raise what ctypes raises, what
ctypes accepts is accepted, and without the extension the binding is the same."""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2510_14126_amd import binding as pa  # noqa: E402

ARGS = {   # a valid no-op call of each function (batch 0), in the C order
    "paged_attn_decode": ["pool", "t", "t", 4, "t", 0, 8, 0.125, 50, 16, "t", "t", "t", None],
    "paged_attn_decode_scheduled": ["pool", "t", "t", 4, "t", 0, 8, 0.125, 50, 16, "t", 0, "t", "t", "t", None],
    "paged_attn_reduce": ["t", "t", "t", 0, 8, 64, 16, 4, "t", None],
    "paged_attn_decode_cascade": ["pool", "t", "t", 4, "t", 0, 8, 0.125, 50, 16, 16, 16, "t", "t", None],
    "paged_attn_decode_cascade_scheduled": ["pool", "t", "t", 4, "t", 0, 8, 0.125, 50, 16, 16, 16, "t", 0, "t", "t",
                                            None],
    "paged_attn_decode_cascade_groups": ["pool", "t", "t", 4, "t", 0, 8, 0.125, 50, 16, 16, 16, "t", 1, 1, 16, "t",
                                         0, "t", "t", None],
    "paged_attn_reduce_cascade": ["t", "t", "t", 0, 8, 64, 16, 16, 16, 4, "t", None],
    "paged_attn_reduce_cascade_groups": ["t", "t", "t", 0, 8, 64, 16, 16, 16, 16, 4, "t", None],
    "paged_attn_append_kv": ["pool", "t", "t", "t", 4, "t", 0, None],
    "paged_attn_decode_append": ["pool", "t", "t", "t", "t", 4, "t", 0, 8, 0.125, 50, 16, "t", 0, "t", "t", "t", None],
    "paged_attn_decode_cascade_append": ["pool", "t", "t", "t", "t", 4, "t", 0, 8, 0.125, 50, 16, 16, 16, "t", 1, 1, 0,
                                         "t", 0, "t", "t", None],
    "paged_attn_decode_noalloc": ["pool", "t", "t", 4, "t", 0, 8, 0.125, 50, 16, "t", None],
    "paged_attn_extend": ["pool", "t", "t", 0, "t", 4, "t", 0, 8, 0.125, 50, 16, "t", None],
}


def test_every_native_call_is_listed():
    assert set(pa._pycall.NAMES) == set(ARGS)


@pytest.mark.parametrize("name", sorted(ARGS))
def test_same_status_as_ctypes(name):
    t = torch.zeros(64, dtype=torch.int32)
    pool = pa.kv_pool_create(4, 16, 2, 128 if "cascade" in name or "extend" in name else 64, t, t)
    fill = {"pool": pool.handle, "t": t}
    args = [fill.get(a, a) if isinstance(a, str) else a for a in ARGS[name]]
    native, plain = getattr(pa._pycall, name), getattr(pa._lib, name)

    def both(a):
        rc = native(*a)
        said = pa.pa_last_error()
        assert rc == plain(*[x.data_ptr() if hasattr(x, "data_ptr") else int(x) if isinstance(x, np.integer) else x
                             for x in a])
        assert rc == pa.PA_OK or said == pa.pa_last_error()
        return rc

    assert both(args) == pa.PA_OK
    assert both([np.int64(a) if type(a) is int else a for a in args]) == pa.PA_OK
    assert both([a.data_ptr() if a is t else a for a in args]) == pa.PA_OK
    refused = 0
    for i, a in enumerate(args):           # one argument at a time: NULL, -1 or NaN
        bad = None if a is t or a is None or ARGS[name][i] == "pool" else float("nan") if type(a) is float else -1
        refused += both(args[:i] + [bad] + args[i + 1:]) != pa.PA_OK
    assert refused >= 2
    with pytest.raises(TypeError):
        native(*args[:-1])
    with pytest.raises(ctypes.ArgumentError):
        native(*[1.5 if type(a) is int else a for a in args])
    pool.close()


# through the public functions, which are the same with and without the extension
FORMS = """
import ctypes, sys
if {hide}:
    sys.modules["paper_2510_14126_amd._pycall"] = None
import torch
from paper_2510_14126_amd import binding as pa
assert hasattr(pa._pycall, "NAMES") == (not {hide})
t = torch.zeros(64, dtype=torch.int32)
pool = pa.kv_pool_create(4, 16, 2, 64, t, t)

class Param:
    def __init__(self, x):
        self._as_parameter_ = x

def said(**kw):
    args = dict(q=t, block_tables=t, bt_stride=4, context_lens=t, batch=0, num_q_heads=8, scale=0.125,
                max_context_len=50, partition_size=16, out=t, partial_out=t, partial_lse=t)
    args.update(kw)
    try:
        pa.paged_attn_decode(pool, **args)
        return "accepted"
    except Exception as e:
        return f"{{type(e).__module__}}.{{type(e).__name__}}: {{e}}"

for kw in (dict(), dict(batch=1.5), dict(batch="1"), dict(batch=None), dict(scale="x"), dict(scale=None),
           dict(scale=ctypes.c_float(0.125)), dict(scale=1), dict(batch=ctypes.c_int32(0)),
           dict(bt_stride=Param(4)), dict(bt_stride=ctypes.c_int32(1)), dict(max_context_len=True), dict(q="12"), dict(q="x"),
           dict(q=[1]), dict(q=1.5), dict(q=2 ** 70), dict(batch=2 ** 40), dict(stream=torch), dict(scale=1e300)):
    print(sorted(kw), said(**kw))
"""


def test_accepts_and_raises_as_ctypes_does():
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = [subprocess.run([sys.executable, "-c", FORMS.format(hide=hide)], cwd=root, capture_output=True, text=True)
           for hide in (False, True)]
    assert out[0].returncode == 0 and out[1].returncode == 0, out[0].stderr + out[1].stderr
    native, plain = (x.stdout.splitlines() for x in out)
    assert native == plain and len(native) == 20
    assert sum("ctypes.ArgumentError" in x for x in native) >= 4
    assert sum(x.endswith("accepted") for x in native) >= 6


def test_build_without_python_headers(tmp_path, monkeypatch):
    """The library builds where the extension cannot be: no stale one is left."""
    from paper_2510_14126_amd import build
    stale = tmp_path / "_pycall.so"
    stale.write_bytes(b"")
    monkeypatch.setattr(build, "PYCALL_PATH", str(stale))
    monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": str(tmp_path)})
    assert build.build_pycall() is False
    assert not stale.exists()
