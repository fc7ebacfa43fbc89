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
        elif c["call"] == "conv":
            s = c["side"]
            rb.rbgp_conv3x3(m, c["dtype"], M, K // 9, N // s // s, s, s, at, at, at, N)
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


def call(w, N, dtype=rb.F32, transposed=False, knobs={}, ldO=0, kind="spmm", side=4):
    M, K = (w.K, w.M) if transposed else (w.M, w.K)
    return {"mask": [w.rows, w.cols, w.row_deg, w.mask_seed], "transposed": transposed, "call": kind, "dtype": dtype, "M": M, "K": K, "N": N,
            "knobs": knobs, "ldO": ldO, "side": side}


def waves_of(name, lds):
    """Waves that a stage list is split over, of a launch of spmm_reg or spmm_reg_bf16: by the LDS of the partial sums."""
    per_tile = 2 if name.startswith("spmm_reg_bf16") and ", 128, " in name else 1   # (pieces of 16 bytes of a lane's row)
    return {0: 1, 8192: 2, 12288: 4}[lds // per_tile]


# VGG19 conv5 (ten stages of 72 steps, 32 lists a tile of 64 columns), layers 9 and 7 at 1/4 (28 stages, as many lists; twelve, 16
# lists), layer 5 at 1/2 and 4096 x 4096 at 1/8 (tile rows with one list): either side of 256, 512, 768 and 1024 lists.
# (workload, columns, dtype, kernel, waves a list, two chains of sums[, call: "conv" of 4 x 4 pixels])
CONV5, L9, L7 = wl.VGG19_CONV5, wl.vgg19_sweep_workload(9, 2, wl.F32), wl.vgg19_sweep_workload(7, 2, wl.F32)
SPLITS = [
    (CONV5, 512, rb.F32, "spmm_reg", 4, False), (CONV5, 513, rb.F32, "spmm_reg", 2, True), (CONV5, 960, rb.F32, "spmm_reg", 2, True),
    (CONV5, 1024, rb.F32, "spmm_reg", 2, False), (CONV5, 1025, rb.F32, "spmm_reg_dual", None, True),
    (CONV5, 1984, rb.F32, "spmm_reg_dual", None, True), (CONV5, 1985, rb.F32, "spmm_reg_dual", None, False),
    (CONV5, 512, rb.BF16_F32ACC, "spmm_reg_bf16", 4, False), (CONV5, 513, rb.BF16_F32ACC, "spmm_reg_bf16", 2, True),
    (CONV5, 1024, rb.BF16_F32ACC, "spmm_reg_bf16", 2, False), (CONV5, 1025, rb.BF16_F32ACC, "spmm_reg_bf16", 1, True),
    (L9, 512, rb.F32, "spmm_reg", 4, False), (L9, 513, rb.F32, "spmm_reg", 2, True), (L9, 1025, rb.F32, "spmm_reg_dual", None, True),
    (L9, 896, rb.F32, "spmm_reg", 2, True, "conv"), (L9, 912, rb.F32, "spmm_reg", 4, False, "conv"), (L9, 960, rb.F32, "spmm_reg", 2, True),
    (L9, 1025, rb.BF16_F32ACC, "spmm_reg_bf16", 4, False), (L9, 1536, rb.BF16_F32ACC, "spmm_reg_bf16", 4, False),
    (L9, 1537, rb.BF16_F32ACC, "spmm_reg_bf16", 1, True),
    (L7, 1536, rb.F32, "spmm_reg", 4, False), (L7, 1536, rb.BF16_F32ACC, "spmm_reg_bf16", 2, True),
    (wl.vgg19_sweep_workload(7, 4, wl.BF16), 1280, rb.BF16_F32ACC, "spmm_reg_bf16", 4, False),
    (wl.vgg19_sweep_workload(5, 1, wl.F32), 2237, rb.F32, "spmm_reg", 2, False), (wl.sdmm4096_table2(1, 2), 181, rb.F32, "spmm_reg", 2, False),
]


@pytest.mark.parametrize("k", range(len(SPLITS)), ids=lambda k: f"{SPLITS[k][0].name}_{SPLITS[k][1]}_{SPLITS[k][2]}_{len(SPLITS[k])}")
def test_waves_of_a_stage_list(launches, k):
    w, N, dtype, kernel, waves, chains, kind = SPLITS[k] if len(SPLITS[k]) == 7 else SPLITS[k] + ("spmm",)
    rc, last, ran = launches([call(w, N, dtype, kind=kind)])[0]
    assert rc == 0 and last == kernel and len(ran) == 1, (rc, last, ran)
    name, lds = ran[0][0], ran[0][4]
    assert name.startswith(kernel + "<") and name.endswith(", 1>") == chains, ran
    assert waves is None or waves_of(name, lds) == waves, ran


# A batch for every kernel of two chains of sums that the networks and SDMM tables reach: (layer, log2 of 1 / density) of VGG19 or a workload,
# columns, dtype, side of the images of a fused convolution (0: lowered)
TWO_CHAINS = [((4, 4), 2365, 0, 0), ((4, 4), 2368, 0, 8), ((1, 2), 7165, 0, 0), ((1, 2), 7168, 0, 32), ((2, 2), 6144, 0, 16), (wl.sdmm4096_table2(0, 4), 145, 0, 0),
              ((9, 1), 555, 0, 0), ((4, 1), 2368, 0, 8), ((8, 4), 589, 0, 0), ((4, 3), 2368, 0, 8), ((9, 4), 573, 0, 0), ((5, 3), 1536, 0, 8), ((2, 2), 6141, 0, 0),
              ((11, 2), 1027, 0, 0), ((4, 4), 4170, 1, 0), ((4, 4), 1203, 1, 0), ((1, 2), 24573, 1, 0), (wl.WRN_G1, 4321, 1, 0), ((2, 2), 9469, 1, 0),
              ((2, 2), 2207, 1, 0), ((11, 1), 521, 1, 0), ((7, 4), 4143, 1, 0), ((8, 4), 589, 1, 0), ((4, 2), 4797, 1, 0), ((8, 2), 589, 1, 0),
              ((8, 1), 592, 1, 4), ((5, 1), 1536, 1, 8)]


def two_chains(k):
    what, N, dtype, side = TWO_CHAINS[k]
    return (wl.vgg19_sweep_workload(*what, dtype) if isinstance(what, tuple) else what), N, dtype, side


def test_batches_in_two_chains_of_sums(launches):
    cases = [two_chains(k) for k in range(len(TWO_CHAINS))]
    ran = launches([call(w, N, dtype, kind="conv" if side else "spmm", side=side) for w, N, dtype, side in cases])
    for k, (rc, last, kernels) in enumerate(ran):
        assert rc == 0 and last in ("spmm_reg", "spmm_reg_dual", "spmm_reg_bf16") and kernels[0][0].endswith(", 1>"), (TWO_CHAINS[k], last, kernels)
    assert len({r[2][0][0] for r in ran}) >= 25, sorted(r[2][0][0] for r in ran)


# knobs whose kernels are those of every split: lists are split until every SIMD has a wave, whatever their stages
@pytest.mark.parametrize("N,waves", [(765, 4), (1024, 2), (1537, 2), (1984, 2)])
@pytest.mark.parametrize("dtype,knobs", [(rb.F32, {rb.TUNE_REGISTER_SETS: 1}), (rb.F32, {rb.TUNE_REGISTER_SETS: 2}), (rb.F32, {rb.TUNE_ROW_GROUPS: 1}),
                                         (rb.BF16_F32ACC, {rb.TUNE_ROW_GROUPS: 1}), (rb.BF16_F32ACC, {rb.TUNE_REGISTER_SETS: 2})])
def test_knobs_of_the_waves_keep_full_splits(launches, dtype, knobs, N, waves):
    rc, last, ran = launches([call(CONV5, N, dtype, knobs=knobs)])[0]
    assert rc == 0 and last == ("spmm_reg_bf16" if dtype else "spmm_reg"), (rc, last)
    assert waves_of(ran[0][0], ran[0][4]) == waves and not ran[0][0].endswith(", 1>"), ran


def test_two_row_groups_by_hand_keep_full_splits(launches):
    """fp32, two tile rows with one list a wave (VGG19 layer 5 at 1/2, 16 stages), 16 lists of two a tile of 64 columns."""
    w = wl.vgg19_sweep_workload(5, 1, wl.F32)
    ran = launches([call(w, N, knobs={rb.TUNE_ROW_GROUPS: 2}) for N in (16 * 64, 25 * 64, 35 * 64)])
    assert [waves_of(r[2][0][0], r[2][0][4] // 2) for r in ran] == [4, 4, 2], ran


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


def test_many_rows_per_tile_and_4_gib_of_rows_of_o(launches):
    """Rows of O of a workgroup of spmm_reg_rows are 32-bit offsets apart up to 4 GiB (288 rows of VGG19 layer 3 at 1/4 transposed, and 512
    bytes), 64-bit ones from there on."""
    w = wl.vgg19_sweep_workload(3, 2, wl.F32)
    last = (2 ** 32 // 4 - 128 - 1) // 288
    near, far = launches([call(w, 3000, transposed=True, ldO=ldO) for ldO in (last, last + 1)])
    assert near[:2] == (0, "spmm_reg_rows<2>") and far[:2] == (0, "spmm_reg_rows<2, 1>"), (near, far)
    assert near[2][0][0] == "spmm_reg_rows<2, 0>" and far[2][0][0] == "spmm_reg_rows<2, 1>" and near[2][0][1:] == far[2][0][1:], (near, far)
