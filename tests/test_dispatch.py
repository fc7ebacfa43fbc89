"""Which kernels a call launches, and how: the library with a stub in the place of the HIP runtime (hip_stub.c), in a child process, on the
CPU.  For rules of the dispatch that results do not show and names alone do not tell apart."""
import json
import os
import re
import subprocess
import sys

import pytest

from paper_2006_13486_amd import binding as rb
from paper_2006_13486_amd import build
from paper_2006_13486_amd import workloads as wl

REPO = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CHILD = """
import ctypes, json, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
stub.stub_take.restype = ctypes.c_char_p
from paper_2006_13486_amd import binding as rb
n, out, at, masks = ctypes.c_int(), [], 1 << 20, {}
for c in json.load(sys.stdin):
    key = json.dumps([c["mask"], c["transposed"]])
    if key not in masks:
        m = rb.rbgp_make_mask(*c["mask"])
        masks[key] = rb.rbgp_mask_transpose(m) if c["transposed"] else m
    m = masks[key]
    knobs = {int(k): v for k, v in c["knobs"].items()}
    for k in range(10):
        rb.rbgp_mask_tune(m, k, knobs.get(k, 0))
    N, M, K = c["N"], c["M"], c["K"]
    ld = -(-N // 8) * 8
    stub.stub_take(ctypes.byref(n))
    try:
        if c["call"] == "spmm":
            rb.rbgp_spmm(m, c["dtype"], M, K, N, at, at, ld, at, c["ldO"] or N)
        else:
            rb.rbgp_sddmm(m, c["dtype"], M, K, N, at, ld, at, ld, at)
        rc = 0
    except rb.RbgpError as e:
        rc = e.code
    ran = stub.stub_take(ctypes.byref(n)).decode().split("\\n")[:-1]
    out.append([rc, rb.rbgp_last_kernel() if rc == 0 else "", [[x.split()[0]] + [int(v) for v in x.split()[1:]] for x in ran]])
json.dump(out, sys.stdout)
"""


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    """A function from calls to (error code, rbgp_last_kernel, [(kernel, grid x, grid y, threads, LDS bytes)])."""
    if not os.path.exists(build.LIB):
        pytest.skip("needs the built library")
    stub = tmp_path_factory.mktemp("stub") / "hip_stub.so"
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-o", str(stub), os.path.join(REPO, "tests", "hip_stub.c")])

    def run(calls):
        env = dict(os.environ, RBGP_NO_TORCH="1", PYTHONPATH=REPO)
        r = subprocess.run([sys.executable, "-c", CHILD, str(stub)], input=json.dumps(calls), capture_output=True, text=True, env=env, cwd=REPO)
        assert r.returncode == 0, r.stderr[-2000:]
        out = json.loads(r.stdout)
        names = sorted({k[0] for _, _, ran in out for k in ran})
        plain = subprocess.check_output(["c++filt"], input="\n".join(names), text=True).splitlines()
        short = {n: re.sub(r"\(anonymous namespace\)::|^void |\([a-z].*", "", p).replace("true", "1").replace("false", "0") for n, p in zip(names, plain)}
        return [(rc, last, [(short[k[0]], *k[1:]) for k in ran]) for rc, last, ran in out]

    return run


def call(w, N, dtype=rb.F32, transposed=False, knobs={}, ldO=0, kind="spmm"):
    M, K = (w.K, w.M) if transposed else (w.M, w.K)
    return {"mask": [w.rows, w.cols, w.row_deg, w.mask_seed], "transposed": transposed, "call": kind, "dtype": dtype, "M": M, "K": K, "N": N,
            "knobs": knobs, "ldO": ldO}


# (mask, columns, partial sums of a value)
FEW_UNITS = [((8, 2, 8, 1), (5, 1, 8, 9), (5, 1, 4, 9)), ((8, 2, 4, 1), (2, 1, 4, 9), (1, 1, 2, 9))]
PARTIAL_SUMS = [(0, 2048, 7), (1, 1024, 8), (1, 3584, 28), (1, 3712, 29), (1, 3968, 31), (1, 4096, 32), (1, 14464, 113), (1, 15000, 118),
                (1, 32768, 128), (1, 131072, 128)]


def test_reducers_by_the_number_of_partial_sums(launches):
    """A thread a value below 8 partial sums, four waves a value below 32, sixteen from there on."""
    ws = [wl.Workload("few_units", *m, 0, rb.F32, 101, 102, 103, 1.0) for m in FEW_UNITS]
    for (k, N, n), (rc, last, ran) in zip(PARTIAL_SUMS, launches([call(ws[k], N, kind="sddmm") for k, N, _ in PARTIAL_SUMS])):
        assert rc == 0 and ran[0][0].startswith("sddmm_reg<") and ran[0][2] == n, (N, n, ran)
        assert [r[0] for r in ran[1:]] == ["sddmm_reduce" if n < 8 else "sddmm_reduce<4>" if n < 32 else "sddmm_reduce<16>"], (N, ran)
        assert last.endswith(" + sddmm_reduce"), last
