"""GPU parity of the backward products (gradients of O = W_s x I for a fixed mask, Section 6)
against the CPU oracle, through the C ABI: dI = W_s^T x dO on the transposed mask, and
dW = (dO x I^T) sampled on the mask."""
from dataclasses import replace

import numpy as np
import pytest

from oracle import rbgp_oracle as orc
from paper_2006_13486_amd import binding as rb
from paper_2006_13486_amd import workloads as wl
from tests import gpu_harness as gh
from tests.test_gpu_parity import FUZZ

pytestmark = pytest.mark.gpu

GEN, MFMA, REG = rb.KERNEL_GENERIC, rb.KERNEL_MFMA, rb.KERNEL_MFMA_REG


def _check_backward(w, N=None, ld_pad=0, kernels=(rb.KERNEL_AUTO,), data=True, weights=True):
    lib, f32 = gh.backward_inputs(w, N)
    dI_ref, dI_den, dW_ref, dW_den = gh.oracle_backward(w, *f32)
    for kernel in kernels:
        if data:
            dI, used = gh.library_spmm_transposed(w, lib[0], lib[2], kernel=kernel, ld_pad=ld_pad)
            err = orc.normalised_error(dI, dI_ref, dI_den)
            print(f"[gpu]   dI kernel {used} normalised error {err:.3e}", flush=True)
            assert err <= gh.TOL[w.dtype], ("dI", w.name, kernel, err)
        if weights:
            dW = gh.library_sddmm(w, lib[2], lib[1], kernel=kernel, ld_pad=ld_pad)
            err = orc.normalised_error(dW, dW_ref, dW_den)
            print(f"[gpu]   dW normalised error {err:.3e}", flush=True)
            assert err <= gh.TOL[w.dtype], ("dW", w.name, kernel, err)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("idx", range(len(FUZZ)))
def test_backward_products_across_the_kernel_table(idx, dtype):
    rows, cols, deg = FUZZ[idx]
    w = wl.Workload(f"bwd{idx}_{dtype}", rows, cols, deg, 328, dtype, 400 + idx, 500 + idx, 600 + idx, 1.0)
    _check_backward(w, kernels=(rb.KERNEL_AUTO, GEN))


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("N,ld_pad", [(1, 7), (15, 1), (16, 0), (33, 3), (200, 8), (1000, 0), (2049, 15)])
def test_backward_products_ragged_batch(N, ld_pad, dtype):
    """Batch sizes around the kernels' column steps (16 / 32 per iteration, ranges of the split),
    odd leading dimensions included (bf16 with an odd one runs on the plain kernel)."""
    w = wl.Workload(f"bwd_ragged_{dtype}", (4, 2, 2, 4), (4, 2, 4, 9), (2, 2, 4, 9), N, dtype, 41, 42, 43, 1.0)
    _check_backward(w, ld_pad=ld_pad)


@pytest.mark.parametrize("w", [wl.TINY, wl.VGG19_CONV5, wl.VGG19_CONV3_BF16], ids=lambda w: w.name)
def test_backward_products_config_full_size(w):
    _check_backward(w)


# a stage in pieces of three and two groups of 16 steps, whole stages of 36 and 48 steps, one row group per unit, units over all
# of G_i, and 80 stage rows of it
LINES_SHAPES = [((4, 2, 4, 2), (4, 2, 8, 9), (2, 2, 4, 9)), ((8, 4, 4, 4), (8, 2, 4, 9), (4, 2, 2, 9)),
                ((4, 4, 2, 4), (4, 6, 4, 4), (2, 6, 2, 4)), ((8, 2, 4, 1), (8, 2, 4, 9), (2, 2, 2, 9)),
                ((8, 1, 2, 1), (8, 5, 4, 4), (2, 5, 2, 4))]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("rows,cols,deg", LINES_SHAPES)
def test_weight_gradient_whole_lines(rows, cols, deg, dtype):
    """Batches from where sddmm_lines starts to several parts of the batch (bf16) or where sddmm_reg takes over (fp32, from 1024
    columns on; bf16 below 128): widths around a step of a wave (32 columns in fp32, 64 in bf16) and of a workgroup (eight of
    them), rows that do not start at 16 bytes."""
    w = wl.Workload(f"lines_{dtype}", rows, cols, deg, 0, dtype, 81, 82, 83, 1.0)
    for N, pad in ((65, 1), (128, 0), (130, 2), (255, 5), (511, 1), (512, 0), (514, 4), (1030, 2), (4160, 0), (8250, 6)):
        lib, f32 = gh.backward_inputs(w, N)
        _, _, ref, den = gh.oracle_backward(w, *f32)
        dW = gh.library_sddmm(w, lib[2], lib[1], ld_pad=pad)
        ran = rb.rbgp_last_kernel()
        if dtype == wl.BF16:
            want = "sddmm_generic" if (N + pad) % 2 else "sddmm_reg" if N < 128 else "sddmm_lines"
        else:
            want = "sddmm_lines" if N < 1024 else "sddmm_reg"
        assert ran.startswith(want + "<") or ran == want, (N, ran)
        assert ("sddmm_reduce" in ran) == (N >= (4160 if dtype == wl.BF16 else 1030)), (N, ran)
        err = orc.normalised_error(dW, ref, den)
        print(f"[gpu]   {ran}: dW normalised error {err:.3e}", flush=True)
        assert err <= 4e-6, (N, pad, err)     # (a chain of at most 1030 fp32 roundings of 2^-24 per wave grows like its root)


# one mask for every sddmm_lines<row groups, step groups, all of G_i>: (dtype, those three, columns, rows, cols, degrees)
LINES_KERNELS = [
    (wl.F32, 1, 1, 0, 505, (4, 1, 1, 1), (4, 1, 1, 9), (2, 1, 1, 9)),
    (wl.F32, 1, 2, 0, 505, (4, 2, 4, 4), (4, 1, 4, 9), (2, 1, 2, 9)),
    (wl.F32, 1, 3, 0, 505, (4, 1, 4, 1), (4, 3, 4, 9), (2, 3, 2, 9)),
    (wl.F32, 2, 1, 0, 1155, (4, 4, 8, 4), (32, 1, 1, 9), (16, 1, 1, 9)),
    (wl.F32, 2, 2, 0, 505, (4, 4, 8, 4), (4, 7, 4, 9), (2, 7, 2, 9)),
    (wl.F32, 2, 3, 0, 1155, (32, 1, 8, 1), (8, 6, 4, 9), (4, 6, 2, 9)),
    (wl.F32, 1, 1, 1, 505, (4, 1, 2, 1), (4, 1, 4, 1), (2, 1, 2, 1)),
    (wl.F32, 1, 2, 1, 505, (4, 1, 4, 1), (4, 1, 2, 9), (2, 1, 1, 9)),
    (wl.F32, 1, 3, 1, 505, (4, 1, 4, 1), (4, 1, 4, 9), (2, 1, 2, 9)),
    (wl.F32, 2, 1, 1, 1155, (4, 1, 8, 2), (128, 1, 4, 1), (128, 1, 2, 1)),
    (wl.F32, 2, 2, 1, 505, (4, 1, 8, 1), (32, 7, 8, 3), (32, 7, 4, 3)),
    (wl.F32, 2, 3, 1, 505, (4, 1, 8, 4), (8, 7, 8, 9), (4, 7, 4, 9)),
    (wl.BF16, 1, 1, 0, 505, (4, 1, 1, 1), (4, 1, 1, 9), (2, 1, 1, 9)),
    (wl.BF16, 1, 2, 0, 505, (4, 2, 4, 4), (4, 1, 4, 9), (2, 1, 2, 9)),
    (wl.BF16, 1, 3, 0, 4199, (4, 1, 4, 1), (4, 3, 4, 9), (2, 3, 2, 9)),
    (wl.BF16, 1, 4, 0, 505, (4, 1, 8, 1), (16, 6, 4, 9), (8, 6, 2, 9)),
    (wl.BF16, 1, 5, 0, 505, (4, 1, 8, 1), (16, 4, 8, 9), (8, 4, 4, 9)),
    (wl.BF16, 2, 1, 0, 505, (4, 4, 8, 4), (32, 1, 1, 9), (16, 1, 1, 9)),
    (wl.BF16, 2, 2, 0, 505, (4, 4, 8, 4), (32, 1, 4, 9), (16, 1, 2, 9)),
    (wl.BF16, 2, 3, 0, 505, (32, 1, 8, 1), (8, 6, 4, 9), (4, 6, 2, 9)),
    (wl.BF16, 2, 4, 0, 505, (32, 1, 8, 1), (16, 6, 4, 9), (8, 6, 2, 9)),
    (wl.BF16, 2, 5, 0, 505, (32, 1, 8, 1), (16, 4, 8, 9), (8, 4, 4, 9)),
    (wl.BF16, 1, 1, 1, 505, (4, 1, 2, 1), (4, 1, 4, 1), (2, 1, 2, 1)),
    (wl.BF16, 1, 2, 1, 505, (4, 1, 4, 1), (4, 1, 2, 9), (2, 1, 1, 9)),
    (wl.BF16, 1, 3, 1, 4199, (4, 1, 4, 1), (4, 1, 4, 9), (2, 1, 2, 9)),
    (wl.BF16, 1, 4, 1, 505, (4, 1, 4, 1), (256, 3, 2, 9), (256, 3, 1, 9)),
    (wl.BF16, 1, 5, 1, 505, (4, 1, 2, 1), (256, 1, 8, 9), (256, 1, 4, 9)),
    (wl.BF16, 2, 1, 1, 505, (4, 1, 8, 2), (128, 1, 4, 1), (128, 1, 2, 1)),
    (wl.BF16, 2, 2, 1, 505, (4, 1, 8, 1), (256, 1, 2, 9), (256, 1, 1, 9)),
    (wl.BF16, 2, 3, 1, 505, (4, 1, 8, 4), (64, 1, 8, 9), (32, 1, 4, 9)),
    (wl.BF16, 2, 4, 1, 505, (4, 1, 8, 1), (256, 3, 2, 9), (256, 3, 1, 9)),
    (wl.BF16, 2, 5, 1, 505, (4, 1, 8, 4), (128, 1, 8, 9), (64, 1, 4, 9)),
]


def _kept_products(w, dO, I):
    """sum_n dO[m][n] I[k][n] of every kept (m, k) in float64, laid out as dW."""
    cols = rb.rbgp_mask_columns(gh.make_mask(w)).reshape(w.M, -1)
    with np.errstate(invalid="ignore"):
        return np.take_along_axis(dO.astype(np.float64) @ I.astype(np.float64).T, cols, axis=1)


@pytest.mark.parametrize("dtype,RB,NB,gi,N,rows,cols,deg", LINES_KERNELS)
def test_weight_gradient_every_kernel_of_whole_lines(dtype, RB, NB, gi, N, rows, cols, deg):
    """On the lowered input, with a ragged last step and rows at odd dwords, and (nine taps) as a convolution of 7 x 8 images."""
    w = wl.Workload("lines", rows, cols, deg, 0, dtype, 91, 92, 93, 1.0)
    images = N // 56
    name = lambda conv: f"sddmm_lines<{RB}, {6 if conv and NB > 3 else NB}, {int(dtype == wl.BF16)}, {conv}, {gi}>" + (" + sddmm_reduce" if N >= 4096 else "")

    def check(got, dO, I, want):
        assert rb.rbgp_last_kernel() == want
        err = orc.normalised_error(got, _kept_products(w, dO, I), _kept_products(w, np.abs(dO), np.abs(I)))
        print(f"[gpu]   {want}: dW normalised error {err:.3e}", flush=True)
        assert err <= 4e-6, (want, err)      # (as test_weight_gradient_whole_lines: chains are no longer)

    lib, f32 = gh.backward_inputs(w, N)
    check(gh.library_sddmm(w, lib[2], lib[1], ld_pad=1 if dtype == wl.BF16 else 2), f32[2], f32[1], name(0))
    if cols[3] != 9:
        return
    X, dO = wl.conv_activations(w, images, 7, 8), wl.output_gradients(w, images * 56)
    if dtype == wl.BF16:
        Xl, dOl = wl.to_bf16_bits(X), wl.to_bf16_bits(dO)
        X, dO = wl.bf16_bits_as_f32(Xl), wl.bf16_bits_as_f32(dOl)
    else:
        Xl, dOl = X, dO
    check(gh.library_conv3x3_sddmm(w, dOl, Xl), dO, orc.im2col_3x3(X), name(1))


# (mask, dtype, side of the images or 0 on the lowered input, columns, padding of the rows, kernel): both sides of the lines
# that the dispatch draws by the batch
ONE_LAUNCH = ((16, 4, 4, 2), (16, 4, 8, 9), (2, 4, 4, 9))     # (one row group per unit)
UNSPLIT = ((4, 4, 4, 2), (8, 2, 4, 9), (4, 2, 2, 9))          # (a workgroup per unit)
TWO_GROUPS = ((8, 4, 4, 2), (8, 4, 8, 9), (4, 4, 8, 9))
HALVED = ((8, 4, 4, 2), (8, 4, 8, 9), (4, 4, 4, 9))           # (bf16: a workgroup per row group; sddmm_reg takes both)
ONE_FULL_GROUP = ((32, 2, 4, 2), (16, 2, 8, 9), (2, 2, 4, 9))
MANY_UNITS = ((32, 4, 32, 1), (32, 1, 32, 1), (16, 1, 8, 1))  # (one step group per stage: eight steps, four, one row per column set)
FOUR_STEPS = ((32, 4, 32, 1), (32, 1, 32, 1), (16, 1, 4, 1))
LONE_ROWS = ((32, 1, 128, 1), (32, 1, 32, 1), (16, 1, 8, 1))
BY_BATCH = [(ONE_LAUNCH, wl.BF16, 0, 512, 0, "lines"), (ONE_LAUNCH, wl.BF16, 0, 960, 0, "reg"), (ONE_LAUNCH, wl.BF16, 0, 1408, 0, "lines"),
            (ONE_LAUNCH, wl.BF16, 0, 1408, 8, "reg"), (ONE_LAUNCH, wl.F32, 0, 256, 0, "lines"), (ONE_LAUNCH, wl.F32, 0, 1024, 0, "reg"),
            (ONE_LAUNCH, wl.F32, 4, 1712, 0, "lines"), (ONE_LAUNCH, wl.F32, 4, 1728, 0, "reg"),
            (UNSPLIT, wl.BF16, 0, 256, 0, "reg"), (UNSPLIT, wl.BF16, 0, 258, 6, "lines"), (UNSPLIT, wl.BF16, 0, 3200, 0, "lines"),
            (UNSPLIT, wl.BF16, 0, 3328, 0, "reg"), (UNSPLIT, wl.BF16, 8, 3328, 0, "lines"), (UNSPLIT, wl.BF16, 0, 16384, 0, "lines"),
            (UNSPLIT, wl.F32, 0, 512, 0, "lines"), (UNSPLIT, wl.F32, 0, 514, 1, "reg"),
            (HALVED, wl.BF16, 0, 24576, 0, "lines"), (HALVED, wl.BF16, 0, 24640, 0, "reg"),
            (HALVED, wl.BF16, 8, 20480, 0, "lines"), (HALVED, wl.BF16, 8, 20544, 0, "reg"),
            (ONE_FULL_GROUP, wl.BF16, 0, 3584, 0, "lines"), (ONE_FULL_GROUP, wl.BF16, 0, 4096, 0, "reg"),
            (MANY_UNITS, wl.BF16, 0, 1536, 0, "lines"), (MANY_UNITS, wl.BF16, 0, 2048, 0, "reg"), (MANY_UNITS, wl.BF16, 0, 2304, 0, "lines"),
            (FOUR_STEPS, wl.BF16, 0, 2048, 0, "lines"), (LONE_ROWS, wl.BF16, 0, 2560, 0, "reg"), (LONE_ROWS, wl.BF16, 0, 3072, 0, "lines"),
            (TWO_GROUPS, wl.F32, 8, 4416, 0, "lines"), (TWO_GROUPS, wl.F32, 8, 4480, 0, "reg"), (TWO_GROUPS, wl.F32, 0, 4480, 3, "lines")]


@pytest.mark.parametrize("mask,dtype,side,N,pad,kernel", BY_BATCH)
def test_weight_gradient_kernel_by_batch(mask, dtype, side, N, pad, kernel):
    w = wl.Workload("by_batch", *mask, 0, dtype, 97, 98, 99, 1.0)
    dO = wl.output_gradients(w, N)
    I = wl.conv_activations(w, N // side ** 2, side, side) if side else wl.activations(w, N)
    bits = wl.to_bf16_bits if dtype == wl.BF16 else lambda x: x
    back = wl.bf16_bits_as_f32 if dtype == wl.BF16 else lambda x: x
    dO_lib, I_lib = bits(dO), bits(I)
    got = gh.library_conv3x3_sddmm(w, dO_lib, I_lib) if side else gh.library_sddmm(w, dO_lib, I_lib, ld_pad=pad)
    assert rb.rbgp_last_kernel().startswith(f"sddmm_{kernel}<")
    dO, I = back(dO_lib), back(I_lib)
    I = orc.im2col_3x3(I) if side else I
    err = orc.normalised_error(got, _kept_products(w, dO, I), _kept_products(w, np.abs(dO), np.abs(I)))
    print(f"[gpu]   {rb.rbgp_last_kernel()}: dW normalised error {err:.3e}", flush=True)
    assert err <= 4e-6


FEW_UNITS = ((4, 4, 8, 4), (28, 1, 8, 9), (14, 1, 4, 9))      # (224 units of one workgroup: partial sums in sddmm_reg only)


@pytest.mark.parametrize("mask_of,dtype,large,small", [(UNSPLIT, wl.F32, 2100, 2048), (UNSPLIT, wl.BF16, 20992, 10240),
                                                       (FEW_UNITS, wl.F32, 2000, 700)])
def test_weight_gradient_of_a_smaller_batch_allocates_nothing(mask_of, dtype, large, small):
    """An eager call on a batch that takes fewer partial sums than a smaller one does, or none, then the capture of the smaller
    one: three replays on fresh inputs against the eager result."""
    import torch
    w = wl.Workload("smaller", *mask_of, 0, dtype, 97, 98, 99, 1.0)
    mask = gh.make_mask(w)
    t = torch.float32 if dtype == wl.F32 else torch.bfloat16
    dO, I = (torch.randn((rows, large), device="cuda:0").to(t) for rows in (w.M, w.K))
    dW = torch.zeros(w.nnz, device="cuda:0")
    call = lambda N: rb.rbgp_sddmm(mask, dtype, w.M, w.K, N, dO.data_ptr(), large, I.data_ptr(), large, dW.data_ptr(),
                                   torch.cuda.current_stream().cuda_stream)
    call(large)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(small)
    assert "sddmm_reduce" in rb.rbgp_last_kernel()
    for _ in range(3):
        dO.copy_(torch.randn(dO.shape, device="cuda:0"))
        call(small)
        torch.cuda.synchronize()
        want = dW.clone()
        dW.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(dW, want)


@pytest.mark.parametrize("case", [c for c in LINES_KERNELS if c[0] == wl.F32 and c[1:4] in ((1, 3, 0), (1, 3, 1), (2, 2, 0))])
def test_weight_gradient_of_a_convolution_keeps_infinities(case):
    """fp32 on split operands with pixels and gradients that are not finite or beyond the range of the split: the second pass
    of the fused form gives the sums of the definition, the other sums stay as they are."""
    _, RB, NB, gi, N, rows, cols, deg = case
    w = wl.Workload("lines_conv_inf", rows, cols, deg, 0, wl.F32, 94, 95, 96, 1.0)
    images = N // 56
    X, dO = wl.conv_activations(w, images, 7, 8), wl.output_gradients(w, images * 56)
    clean = gh.library_conv3x3_sddmm(w, dO, X)
    assert rb.rbgp_last_kernel() == f"sddmm_lines<{RB}, {NB}, 0, 1, {gi}>"
    bad, dO_bad = X.copy(), dO.copy()
    bad[1, 0, 0, 0], bad[2, images - 1, 6, 7], bad[0, 1, 3, 4] = np.inf, np.nan, np.float32(2.0 ** 106)
    dO_bad[1, 60], dO_bad[2, images * 56 - 1] = -np.inf, np.float32(2.0 ** 107)
    got = gh.library_conv3x3_sddmm(w, dO_bad, bad)
    I = orc.im2col_3x3(bad)
    ref, size = _kept_products(w, dO_bad, I), _kept_products(w, np.abs(dO_bad), np.abs(I))
    # (a product of two operands near the top of fp32 leaves its range)
    over = np.abs(ref) > np.finfo(np.float32).max
    ref[over] = np.sign(ref[over]) * np.inf
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(got == np.inf, ref == np.inf) and np.array_equal(got == -np.inf, ref == -np.inf)
    fin = np.isfinite(ref)
    assert fin.any() and not fin.all() and (np.abs(got[fin] - ref[fin]) <= 4e-6 * size[fin]).all()
    kept = rb.rbgp_mask_columns(gh.make_mask(w)).reshape(w.M, -1)
    same = ~np.any(I != orc.im2col_3x3(X), axis=1)[kept] & ~np.any(dO_bad != dO, axis=1)[:, None]
    assert same.any() and np.array_equal(got[same], clean[same])


# fp32 convolutions whose units do not fill the chip: (mask, images of 8 x 8 pixels, kernel)
BATCH_IN_PARTS = [(((8, 4, 4, 2), (4, 4, 8, 9), (2, 4, 4, 9)), 17, "1, 3, 0, 1, 0"), (((8, 4, 4, 2), (4, 4, 8, 9), (2, 4, 4, 9)), 97, "2, 3, 0, 1, 0"),
                  (((8, 2, 4, 1), (8, 2, 4, 9), (2, 2, 2, 9)), 33, "1, 3, 0, 1, 1"), (((4, 4, 4, 2), (8, 2, 4, 9), (4, 2, 2, 9)), 65, "1, 3, 0, 1, 0")]


@pytest.mark.parametrize("mask,images,kernel", BATCH_IN_PARTS)
def test_weight_gradient_of_a_convolution_in_parts_of_the_batch(mask, images, kernel):
    """Partial sums of parts with a ragged last step, one of them with an infinite pixel."""
    w = wl.Workload("parts", *mask, 0, wl.F32, 101, 102, 103, 1.0)
    X, dO = wl.conv_activations(w, images, 8, 8), wl.output_gradients(w, images * 64)
    X[1, images - 1, 7, 7] = np.inf
    got = gh.library_conv3x3_sddmm(w, dO, X)
    assert rb.rbgp_last_kernel() == f"sddmm_lines<{kernel}> + sddmm_reduce"
    I = orc.im2col_3x3(X)
    ref, size = _kept_products(w, dO, I), _kept_products(w, np.abs(dO), np.abs(I))
    fin = np.isfinite(ref)
    assert fin.any() and not fin.all() and np.array_equal(np.isfinite(got), fin)
    assert (np.abs(got[fin] - ref[fin]) <= 4e-6 * size[fin]).all()   # (as test_weight_gradient_whole_lines: chains are no longer)


@pytest.mark.parametrize("dtype,images", [(wl.BF16, 32771), (wl.F32, 16387)])
@pytest.mark.parametrize("mask", [((8, 2, 4, 1), (2, 2, 4, 9), (2, 2, 2, 9)), ((8, 2, 4, 1), (4, 1, 4, 9), (2, 1, 4, 9))])
def test_weight_gradient_of_a_convolution_with_gradients_beyond_4_gib(mask, dtype, images):
    """Rows of dO past 4 GiB: gradients in some columns at both ends and between, zeros elsewhere."""
    import torch
    w = wl.Workload("far", *mask, 0, dtype, 107, 108, 109, 1.0)
    t, side, C = torch.float32 if dtype == wl.F32 else torch.bfloat16, 32, w.K // 9
    N = images * side * side
    g = torch.Generator(device="cuda:0").manual_seed(1)
    X = torch.zeros((C, images, side + 2, side + 2), dtype=t, device="cuda:0")
    X[:, :, 1:-1, 1:-1] = torch.randn((C, images, side, side), generator=g, device="cuda:0").to(t)
    dO = torch.zeros((w.M, N), dtype=t, device="cuda:0")
    assert dO.numel() * dO.element_size() > 2 ** 32 and X.numel() * X.element_size() < 2 ** 31
    at = torch.cat([torch.arange(70), torch.randint(70, N - 70, (400,), generator=torch.Generator().manual_seed(2)).unique(), torch.arange(N - 70, N)]).cuda()
    dO[:, at] = torch.randn((w.M, at.numel()), generator=g, device="cuda:0").to(t)
    mask_ = gh.make_mask(w)
    dW = torch.full((w.nnz,), float("nan"), device="cuda:0")
    rb.rbgp_conv3x3_sddmm(mask_, dtype, w.M, C, images, side, side, dO.data_ptr(), N, X.data_ptr(), dW.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rb.rbgp_last_kernel() == f"sddmm_lines<{1 if mask[1][1] == 2 else 2}, 3, {int(dtype == wl.BF16)}, 1, 0, 1> + sddmm_reduce"
    img, y, x = at // side ** 2, at % side ** 2 // side, at % side
    I = torch.stack([X[:, img, y + dy, x + dx] for dy in range(3) for dx in range(3)], 1).reshape(w.K, -1).double()   # row 9 c + tap
    kept = torch.from_numpy(rb.rbgp_mask_columns(mask_).reshape(w.M, -1)).long().cuda()
    take = lambda a, b: torch.gather(a @ b.T, 1, kept).reshape(-1)
    d = dO[:, at].double()
    assert bool(((dW.double() - take(d, I)).abs() <= 4e-6 * take(d.abs(), I.abs())).all())


@pytest.mark.parametrize("N", [130, 200])
def test_weight_gradient_split_operands_keep_infinities_and_tiny_operands(N):
    """fp32 weight gradients on split operands against the plain kernel: the same sums are infinite or not a number, operands
    beyond bf16's largest number give finite sums, rows down to fp32's denormals lose nothing."""
    w = wl.Workload("lines_inf", (4, 2, 4, 2), (4, 2, 8, 9), (2, 2, 4, 9), 0, wl.F32, 84, 85, 86, 1.0)
    lib, _ = gh.backward_inputs(w, N)
    I, dO = lib[1].copy(), lib[2].copy()
    clean = gh.library_sddmm(w, dO, I)
    I[5, 7], I[40, N - 1], dO[3, 20], dO[9, 21] = np.inf, np.nan, -np.inf, np.float32(1e37)
    got, ref = gh.library_sddmm(w, dO, I), gh.library_sddmm(w, dO, I, kernel=GEN)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
    fin = np.isfinite(ref)
    rows = np.ones(w.M, bool)
    rows[[3, 9]] = False
    assert np.allclose(got[9][fin[9]], ref[9][fin[9]], rtol=1e-5)
    same = fin & rows[:, None]
    assert np.array_equal(got[same], clean[same])
    scale = 2.0 ** np.random.default_rng(7).choice([0, -40, -100, -118, -130], (w.M, 1))
    tiny = (lib[2] * scale).astype(np.float32)
    got = gh.library_sddmm(w, tiny, lib[1])
    cols = rb.rbgp_mask_columns(gh.make_mask(w)).reshape(w.M, -1)
    X, D = lib[1].astype(np.float64), tiny.astype(np.float64)
    exact = np.stack([X[cols[m]] @ D[m] for m in range(w.M)])
    size = np.stack([np.abs(X[cols[m]]) @ np.abs(D[m]) for m in range(w.M)])
    assert (np.abs(got - exact) <= (N + 8) * (2.0 ** -24 * size + 2.0 ** -150)).all()


def test_weight_gradient_wrn_full_batch():
    """131072 columns: the batch is cut into many ranges whose partial sums are added in a second kernel."""
    _check_backward(wl.WRN_G1, data=False)


def test_backward_data_product_wrn_sampled_batch():
    _check_backward(replace(wl.WRN_G1, N=4096), weights=False)


def test_weight_gradient_repeated_calls_and_growing_batch():
    """The partial-sum buffer is kept with the mask: a small batch first, then a larger one, then the
    small one again, every result checked."""
    mask_w = wl.Workload("bwd_grow", (4, 2, 4, 2), (4, 2, 8, 9), (2, 2, 4, 9), 0, wl.F32, 51, 52, 53, 1.0)
    for N in (96, 4000, 96):
        _check_backward(replace(mask_w, N=N), data=False)


def test_weight_gradient_empty_batch_stores_zeros():
    w = replace(wl.TINY, N=0)
    dW = gh.library_sddmm(w, np.zeros((w.M, 0), np.float32), np.zeros((w.K, 0), np.float32))
    assert not dW.any()


@pytest.mark.parametrize("kernel", [rb.KERNEL_AUTO, GEN])
def test_weight_gradient_one_hot_inputs_are_exact(kernel):
    """dO = ones in column n of every row, I = distinct powers of two in the same column: dW repeats
    the value of I at each kept column exactly."""
    w = replace(wl.TINY, N=40)
    dO = np.zeros((w.M, w.N), np.float32); dO[:, 17] = 1.0
    I = np.zeros((w.K, w.N), np.float32); I[:, 17] = np.ldexp(1.0, np.arange(w.K) % 24 - 12).astype(np.float32)
    I[:, 3] = 5.0                                   # a column that dO does not touch
    dW = gh.library_sddmm(w, dO, I, kernel=kernel)
    mask = rb.rbgp_make_mask(w.rows, w.cols, w.row_deg, w.mask_seed)
    cols = rb.rbgp_mask_columns(mask).reshape(w.M, w.rowdeg)
    assert np.array_equal(dW, I[cols, 17])


def test_masks_outside_rbgp4_roles_take_the_plain_kernels():
    w = wl.Workload("bwd_sparse_gr", (4, 4, 4, 2), (4, 4, 4, 2), (2, 2, 2, 2), 100, wl.F32, 1, 2, 3, 1.0)
    _check_backward(w)


def test_weight_gradient_bf16_odd_leading_dimension():
    w = wl.Workload("bwd_odd_ld", (4, 2, 2, 4), (4, 2, 4, 9), (2, 2, 4, 9), 77, wl.BF16, 44, 45, 46, 1.0)
    _check_backward(w, data=False)


def test_pack_transposed_from_device_values_matches_host_values():
    """The same kept values, resident on the device in the forward mask's order, packed for both products."""
    import torch
    w = wl.Workload("bwd_devpack", (4, 2, 4, 2), (4, 2, 8, 9), (2, 2, 4, 9), 64, wl.F32, 54, 55, 56, 1.0)
    mask = gh.make_mask(w)
    mask_t = rb.rbgp_mask_transpose(mask)
    vals = wl.kept_weights(w).reshape(-1)
    stream = torch.cuda.current_stream().cuda_stream
    nbytes = rb.rbgp_packed_bytes(mask_t, w.dtype)
    a = torch.zeros(nbytes, dtype=torch.uint8, device="cuda:0")
    b = torch.zeros(nbytes, dtype=torch.uint8, device="cuda:0")
    rb.rbgp_pack_transposed(mask_t, w.dtype, vals, a.data_ptr(), stream)
    vals_d = torch.from_numpy(vals).to("cuda:0")
    rb.rbgp_pack_transposed_device(mask_t, w.dtype, vals_d.data_ptr(), b.data_ptr(), stream)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    # and it is the transposed mask's own packing of the reordered values
    c = torch.zeros(nbytes, dtype=torch.uint8, device="cuda:0")
    rb.rbgp_pack(mask_t, w.dtype, np.ascontiguousarray(vals[rb.rbgp_transpose_order(mask)]), c.data_ptr(), stream)
    torch.cuda.synchronize()
    assert torch.equal(a, c)


# ------------------------------------------------------------------ weight gradient of the fused 3x3 convolution
CONV_GRAD_CASES = [
    # workload (K = 9 * channels), images, height, width
    (wl.Workload("cgrad_small", (4, 2, 2, 4), (4, 2, 4, 9), (2, 2, 4, 9), 0, wl.F32, 61, 62, 63, 1.0), 3, 4, 8),
    (wl.Workload("cgrad_ragged", (4, 1, 4, 3), (4, 2, 4, 9), (2, 2, 2, 9), 0, wl.F32, 64, 65, 66, 1.0), 5, 3, 4),
    (wl.Workload("cgrad_wide", (4, 2, 4, 1), (4, 2, 4, 9), (2, 2, 2, 9), 0, wl.F32, 67, 68, 69, 1.0), 2, 5, 32),
    (wl.Workload("cgrad_pad54", (4, 2, 4, 1), (4, 1, 12, 9), (2, 1, 6, 9), 0, wl.F32, 74, 75, 76, 1.0), 2, 4, 8),
    (wl.Workload("cgrad_bf16", (4, 2, 2, 4), (4, 2, 4, 9), (2, 2, 4, 9), 0, wl.BF16, 71, 72, 73, 1.0), 3, 5, 8),
    (wl.Workload("cgrad_bf16_wide", (4, 2, 4, 1), (4, 2, 4, 9), (2, 2, 2, 9), 0, wl.BF16, 77, 78, 79, 1.0), 7, 3, 16),
    (wl.VGG19_CONV5, 128, 4, 4),                                        # the headline layer
    (replace(wl.VGG19_CONV3_BF16, name="cgrad_conv3_bf16"), 128, 8, 8),
    (replace(wl.WRN_G1, name="cgrad_wrn_batch8"), 8, 32, 32),
]


@pytest.mark.parametrize("case", CONV_GRAD_CASES, ids=lambda c: c[0].name)
def test_fused_conv3x3_weight_gradient_equals_sddmm_on_the_lowered_input(case):
    w, B, H, W = case
    w = replace(w, N=B * H * W)
    X = wl.conv_activations(w, B, H, W)
    dO = wl.output_gradients(w)
    if w.dtype == wl.BF16:
        Xl, dOl = wl.to_bf16_bits(X), wl.to_bf16_bits(dO)
        X, dO = wl.bf16_bits_as_f32(Xl), wl.bf16_bits_as_f32(dOl)
    else:
        Xl, dOl = X, dO
    got = gh.library_conv3x3_sddmm(w, dOl, Xl)
    Bs, _ = orc.sample_factors(w.rows, w.cols, w.row_deg, w.mask_seed)
    mask = orc.kron_mask(Bs)
    I = orc.im2col_3x3(X)
    ref, den = orc.sddmm_definition(mask, dO, I), orc.sddmm_definition(mask, np.abs(dO), np.abs(I))
    err = orc.normalised_error(got, ref, den)
    print(f"[gpu]   normalised error {err:.3e}", flush=True)
    assert err <= gh.TOL[w.dtype], err


def test_fused_conv3x3_weight_gradient_argument_checks():
    w = wl.Workload("cgrad_args", (4, 2, 2, 4), (4, 2, 4, 9), (2, 2, 4, 9), 0, wl.F32, 1, 2, 3, 1.0)
    mask = gh.make_mask(w)
    lib = rb.load()
    C = w.K // 9
    assert lib.rbgp_conv3x3_sddmm(mask.handle, 0, w.M, C, 2, 4, 6, 256, 48, 256, 256, None) == rb.ESHAPE      # width % 4
    assert lib.rbgp_conv3x3_sddmm(mask.handle, 1, w.M, C, 2, 4, 4, 256, 32, 256, 256, None) == rb.ESHAPE      # bf16: width % 8
    assert lib.rbgp_conv3x3_sddmm(mask.handle, 0, w.M, C + 1, 2, 4, 4, 256, 32, 256, 256, None) == rb.ESHAPE
    assert lib.rbgp_conv3x3_sddmm(mask.handle, 0, w.M, C, 2, 4, 4, 256, 16, 256, 256, None) == rb.ESHAPE      # ld_dO < N
    assert lib.rbgp_conv3x3_sddmm(mask.handle, 0, w.M, C, 2, 4, 4, 256, 32, None, 256, None) == rb.EINVAL
    tiny = gh.make_mask(wl.TINY)                                                                             # |G_b.V| != 9
    assert lib.rbgp_conv3x3_sddmm(tiny.handle, 0, wl.TINY.M, wl.TINY.K // 9, 1, 1, 4, 256, 4, 256, 256, None) in (rb.ESHAPE, rb.EUNSUPPORTED)


# ------------------------------------------------------------------ gradient of the fused convolution w.r.t. its input
@pytest.mark.parametrize("case", CONV_GRAD_CASES, ids=lambda c: c[0].name)
def test_fused_conv3x3_input_gradient_is_the_transposed_convolution(case):
    w, B, H, W = case
    w = replace(w, N=B * H * W)
    vals, dO = wl.kept_weights(w), wl.output_gradients(w)
    if w.dtype == wl.BF16:
        vl, dOl = wl.to_bf16_bits(vals), wl.to_bf16_bits(dO)
        vals, dO = wl.bf16_bits_as_f32(vl), wl.bf16_bits_as_f32(dOl)
    else:
        vl, dOl = vals, dO
    got, used = gh.library_conv3x3_input_gradient(w, vl, dOl, B, H, W)
    assert used == REG
    Bs, _ = orc.sample_factors(w.rows, w.cols, w.row_deg, w.mask_seed)
    mask = orc.kron_mask(Bs)
    Wd = orc.scatter_values(mask, vals)
    maskT, WT = np.ascontiguousarray(mask.T), np.ascontiguousarray(Wd.T)
    from oracle import naive_c
    dI, dI_den = naive_c.spmm(maskT, WT, dO), naive_c.spmm_abs(maskT, WT, dO)
    ref = orc.col2im_3x3(dI, B, H, W).reshape(w.K // 9, -1)
    den = orc.col2im_3x3(dI_den, B, H, W).reshape(w.K // 9, -1)
    err = orc.normalised_error(got, ref, den)
    print(f"[gpu]   normalised error {err:.3e}", flush=True)
    assert err <= gh.TOL[w.dtype], err


def test_training_step_replays_from_a_hip_graph():
    """Forward, input gradient and weight gradient of a fused 3x3 layer captured into one graph after a
    warm-up call (which builds the library's tables and its partial-sum buffer): three replays on fresh
    inputs, with eager work and synchronisations in between, each compared with the eager result."""
    import torch
    w = wl.Workload("graph_layer", (4, 2, 4, 2), (4, 2, 8, 9), (2, 2, 4, 9), 0, wl.F32, 31, 32, 33, 1.0)
    B, H, W = 6, 8, 8
    N = B * H * W
    C = w.K // 9
    mask = gh.make_mask(w)
    mask_x = rb.rbgp_mask_conv3x3_transpose(mask)
    vals = wl.kept_weights(w).reshape(-1)
    dev = "cuda:0"
    packed = torch.zeros(rb.rbgp_packed_bytes(mask, w.dtype), dtype=torch.uint8, device=dev)
    packed_x = torch.zeros(rb.rbgp_packed_bytes(mask_x, w.dtype), dtype=torch.uint8, device=dev)
    st0 = torch.cuda.current_stream().cuda_stream
    rb.rbgp_pack(mask, w.dtype, vals, packed.data_ptr(), st0)
    rb.rbgp_pack_transposed(mask_x, w.dtype, vals, packed_x.data_ptr(), st0)
    X = torch.zeros(C, B, H + 2, W + 2, device=dev)
    dO = torch.zeros(w.M, B, H + 2, W + 2, device=dev)          # padded: read by the input-gradient convolution
    dO_flat = torch.zeros(w.M, N, device=dev)                   # the same values as a matrix: read by the weight gradient
    O = torch.zeros(w.M, N, device=dev)
    dX = torch.zeros(C, N, device=dev)
    dW = torch.zeros(w.M * w.rowdeg, device=dev)

    def step(stream):
        rb.rbgp_conv3x3(mask, w.dtype, w.M, C, B, H, W, packed.data_ptr(), X.data_ptr(), O.data_ptr(), N, stream)
        rb.rbgp_conv3x3(mask_x, w.dtype, C, w.M, B, H, W, packed_x.data_ptr(), dO.data_ptr(), dX.data_ptr(), N, stream)
        rb.rbgp_conv3x3_sddmm(mask, w.dtype, w.M, C, B, H, W, dO_flat.data_ptr(), N, X.data_ptr(), dW.data_ptr(), stream)

    def fresh_inputs(seed):
        g = torch.Generator(device=dev).manual_seed(seed)
        X[:, :, 1:-1, 1:-1] = torch.randn(C, B, H, W, device=dev, generator=g)
        d = torch.randn(w.M, B, H, W, device=dev, generator=g)
        dO[:, :, 1:-1, 1:-1] = d
        dO_flat.copy_(d.reshape(w.M, N))

    fresh_inputs(0)
    step(st0)                                                    # warm-up: tables, partial sums
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step(torch.cuda.current_stream().cuda_stream)
    for seed in (1, 2, 3):
        fresh_inputs(seed)
        step(torch.cuda.current_stream().cuda_stream)            # eager reference
        torch.cuda.synchronize()
        ref = [t.clone() for t in (O, dX, dW)]
        for t in (O, dX, dW):
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for got, want in zip((O, dX, dW), ref):
            assert torch.equal(got, want)                        # same kernels, same order of sums: bit-identical
