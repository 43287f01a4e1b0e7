"""The native calls of the per-step functions give what ctypes gives: the same
status and message for the same arguments (no GPU: every call here is refused
or is a no-op), for pointers as None, integers and tensors, and for integers
that are not Python ints; wrong counts and types raise."""
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
    with pytest.raises(TypeError):
        native(*[1.5 if type(a) is int else a for a in args])
    pool.close()
