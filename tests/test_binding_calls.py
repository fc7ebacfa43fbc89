"""The binding's calls without ctypes against its ctypes functions: the same calls accepted, refused and reported, on the CPU (no call
reaches a launch: the library returns before one, for N = 0 or with an error)."""
import inspect
import os
import shutil
import sysconfig

import numpy as np
import pytest

from paper_2006_13486_amd import binding as rb
from paper_2006_13486_amd import build
from paper_2006_13486_amd import workloads as wl

CAN_BUILD = shutil.which(os.environ.get("CC", "gcc")) and os.path.exists(os.path.join(sysconfig.get_paths()["include"], "Python.h"))


def test_built_with_the_library_for_this_interpreter():
    if not (os.path.exists(build.LIB) and CAN_BUILD):
        pytest.skip("the library is not built, or this interpreter has no compiler and headers")
    assert rb._call is not None
    assert rb._call.__file__ == build.CALL and build.CALL.endswith(sysconfig.get_config_var("EXT_SUFFIX"))


@pytest.mark.skipif(not CAN_BUILD, reason="no compiler and headers")
def test_a_failed_compile_leaves_no_older_file(tmp_path, monkeypatch, capfd):
    out = tmp_path / os.path.basename(build.CALL)
    (tmp_path / "_call.so").write_bytes(b"older")
    assert build.build_call(str(out)) and [p.name for p in tmp_path.iterdir()] == [out.name]
    monkeypatch.setenv("CC", "/nowhere/cc")
    assert not build.build_call(str(out)) and not list(tmp_path.iterdir())
    assert "ctypes" in capfd.readouterr().err


M = K = 64
PLAIN = {   # every argument after the mask, of a call that the library answers without a GPU
    "rbgp_pack_device": (0, 0, 0),                           # null pointers: EINVAL
    "rbgp_pack_transposed_device": (0, 0, 0),
    "rbgp_spmm": (0, M, K, 0, 1, 1, 0, 1, 0),                # no columns: nothing to do
    "rbgp_sddmm": (0, M, K, 5, 1, 4, 1, 8, 1),               # leading dimension below N: ESHAPE
    "rbgp_conv3x3": (0, M, 7, 1, 4, 4, 1, 1, 1, 16),         # not this mask's channels: ESHAPE
    "rbgp_conv3x3_sddmm": (0, M, 7, 1, 4, 4, 1, 16, 1, 1),
}


@pytest.fixture(scope="module")
def mask():
    rb.load()
    return rb.rbgp_make_mask(wl.TINY.rows, wl.TINY.cols, wl.TINY.row_deg, wl.TINY.mask_seed)


def outcome(fn, *args, **kwargs):
    try:
        return fn(*args, **kwargs)
    except Exception as e:
        return type(e), str(e).replace("_ctypes_", "_"), getattr(e, "code", None)


@pytest.mark.skipif(rb._call is None, reason="csrc/rbgp_call.c is not built")
@pytest.mark.parametrize("name", PLAIN)
def test_same_outcome_as_through_ctypes(mask, name):
    fast, slow, args = getattr(rb, name), rb._WITH_CTYPES[name], PLAIN[name]
    assert fast is not slow
    assert list(inspect.signature(fast).parameters) == list(inspect.signature(slow).parameters)
    assert inspect.signature(fast).parameters["stream"].default == inspect.signature(slow).parameters["stream"].default == 0
    freed = rb.rbgp_make_mask(wl.TINY.rows, wl.TINY.cols, wl.TINY.row_deg, wl.TINY.mask_seed)
    rb.rbgp_mask_free(freed)
    calls = [(mask,) + args, (mask,) + args + (0,), (mask,) + args[:-1], (mask,) + args + (0, 0), (), (None,) + args, (freed,) + args,
             (mask.handle,) + args]
    odd = [True, 1.5, None, "1", np.int64(3), 2**31, -1, -2**63, 2**63, 2**64 + 1, 10**30]
    calls += [(mask,) + args[:k] + (v,) + args[k + 1:] for k in range(len(args)) for v in odd
              if not (name == "rbgp_spmm" and k == 3)]       # (another N of rbgp_spmm would be a launch)
    for c in calls:
        assert outcome(fast, *c) == outcome(slow, *c), (name, c)
    names = list(inspect.signature(slow).parameters)
    assert outcome(fast, mask, **dict(zip(names[1:], args))) == outcome(slow, mask, **dict(zip(names[1:], args)))
    assert outcome(fast, mask, *args, stream=0) == outcome(slow, mask, *args, stream=0)
    assert outcome(fast, mask, *args, nothing=0) == outcome(slow, mask, *args, nothing=0)
