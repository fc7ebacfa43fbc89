"""Batches around the counts at which stage lists are split in four, in two, or walked whole: sums as in 64 bits, whatever the split."""
import pytest
import torch

from paper_2006_13486_amd import binding as rb
from paper_2006_13486_amd import workloads as wl
from tests.test_dispatch import TWO_CHAINS, two_chains

pytestmark = pytest.mark.gpu

# conv5 and VGG19 layer 9 at 1/4, ten and 28 stages: 32 lists a tile of 64 columns.  fp32 and bf16, last columns just inside and just past a
# tile, at 256, 512, 768 and 1024 lists of conv5.  (test_dispatch.py names the kernels and splits)
CONV5 = [c for tiles in (8, 16, 24, 32) for c in (64 * tiles - 3, 64 * tiles + 1)]
CASES = [(wl.VGG19_CONV5, n, dtype) for n in CONV5 for dtype in (rb.F32, rb.BF16_F32ACC)]
CASES += [(wl.vgg19_sweep_workload(9, 2, wl.F32), n, dtype) for n in (253, 513, 765, 769, 1021, 1025, 1535, 1537) for dtype in (rb.F32, rb.BF16_F32ACC)]
# tile rows with one list: 560 and 768 lists in two
CASES += [(wl.vgg19_sweep_workload(5, 1, wl.F32), 2237, rb.F32), (wl.sdmm4096_table2(1, 2), 181, rb.F32)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0].name}_{c[1]}_{c[2]}")
def test_splits_of_stage_lists(case):
    w, N, dtype = case
    t_in = torch.float32 if dtype == rb.F32 else torch.bfloat16
    print(f"[gpu] stage list split {w.name} N={N} dtype={dtype}", flush=True)
    mask = rb.rbgp_make_mask(w.rows, w.cols, w.row_deg, w.mask_seed)
    gen = torch.Generator(device="cuda").manual_seed(11)
    weights = (torch.randn(w.nnz, generator=gen, device="cuda") * w.w_std).to(t_in)
    packed = torch.zeros(rb.rbgp_packed_bytes(mask, dtype), dtype=torch.uint8, device="cuda")
    rb.rbgp_pack_device(mask, dtype, weights.data_ptr(), packed.data_ptr())
    ldI = -(-N // 8) * 8
    I = torch.randn((w.K, ldI), generator=gen, device="cuda").to(t_in)
    out = torch.full((w.M + 1, N), -77.0, device="cuda")
    rb.rbgp_spmm(mask, dtype, w.M, w.K, N, packed.data_ptr(), I.data_ptr(), ldI, out.data_ptr(), N)
    torch.cuda.synchronize()
    assert rb.rbgp_last_kernel().startswith("spmm_reg"), rb.rbgp_last_kernel()
    assert (out[w.M] == -77).all()
    cols = torch.from_numpy(rb.rbgp_mask_columns(mask).reshape(w.M, -1).astype("int64")).cuda()
    dense = torch.zeros((w.M, w.K), dtype=torch.float64, device="cuda").scatter_(1, cols, weights.view(w.M, -1).double())
    I64 = I[:, :N].double()
    bound = cols.shape[1] * 2.0 ** -24 * (dense.abs() @ I64.abs())   # (one fp32 rounding per product and sum, in any order)
    assert bool(((out[:w.M].double() - dense @ I64).abs() <= bound).all())


# (workload, columns, dtype, waves a list that fill every SIMD): one wave, or two, in their place, and paired tile rows
CHAINS = [(wl.VGG19_CONV5, 765, rb.F32, 4), (wl.VGG19_CONV5, 765, rb.BF16_F32ACC, 4), (wl.VGG19_CONV5, 1537, rb.BF16_F32ACC, 2),
          (wl.VGG19_CONV3_BF16, 4000, rb.BF16_F32ACC, 2), (wl.vgg19_sweep_workload(9, 1, wl.F32), 913, rb.F32, 4),
          (wl.vgg19_sweep_workload(4, 4, wl.F32), 3072, rb.F32, 2), (wl.vgg19_sweep_workload(7, 3, wl.F32), 3072, rb.F32, 2),
          (wl.vgg19_sweep_workload(5, 2, wl.F32), 2368, rb.F32, 2)]


@pytest.mark.parametrize("case", CHAINS, ids=lambda c: f"{c[0].name}_{c[1]}_{c[2]}")
def test_fewer_waves_a_list_have_no_longer_chains(case):
    """Where fewer waves take a list than fill every SIMD, the error against 64-bit sums is that of as many waves as do (the same chains
    of fp32 sums, whose totals meet in another order) or less."""
    w, N, dtype, S = case
    t_in = torch.float32 if dtype == rb.F32 else torch.bfloat16
    print(f"[gpu] chains {w.name} N={N} dtype={dtype}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(12)
    weights = (torch.randn(w.nnz, generator=gen, device="cuda") * w.w_std).to(t_in)
    ldI = -(-N // 8) * 8
    I = torch.randn((w.K, ldI), generator=gen, device="cuda").to(t_in)
    mask = rb.rbgp_make_mask(w.rows, w.cols, w.row_deg, w.mask_seed)
    packed = torch.zeros(rb.rbgp_packed_bytes(mask, dtype), dtype=torch.uint8, device="cuda")
    rb.rbgp_pack_device(mask, dtype, weights.data_ptr(), packed.data_ptr())
    cols = torch.from_numpy(rb.rbgp_mask_columns(mask).reshape(w.M, -1).astype("int64")).cuda()
    dense = torch.zeros((w.M, w.K), dtype=torch.float64, device="cuda").scatter_(1, cols, weights.view(w.M, -1).double())
    want = dense @ I[:, :N].double()
    out = torch.empty((w.M, N), device="cuda")

    def error(split):
        rb.rbgp_mask_tune(mask, rb.TUNE_K_SPLIT, split)
        out.fill_(float("nan"))
        rb.rbgp_spmm(mask, dtype, w.M, w.K, N, packed.data_ptr(), I.data_ptr(), ldI, out.data_ptr(), N)
        torch.cuda.synchronize()
        return float((out.double() - want).norm() / want.norm())

    filled, default = error(S), error(0)
    print(f"[gpu]   {default:.3e}, {S} waves a list {filled:.3e}", flush=True)
    # (at least 40 chains' totals of as many products each: another order of the last two or four additions moves the norm by below 2 %)
    assert default <= 1.02 * filled


@pytest.mark.parametrize("k", range(len(TWO_CHAINS)))
def test_two_chains_of_sums(k):
    """Every kernel of two chains, lowered with a ragged last tile and fused, against sums in 64 bits."""
    w, N, dtype, side = two_chains(k)
    t_in = torch.float32 if dtype == rb.F32 else torch.bfloat16
    print(f"[gpu] two chains {w.name} N={N} dtype={dtype} side={side}", flush=True)
    mask = rb.rbgp_make_mask(w.rows, w.cols, w.row_deg, w.mask_seed)
    gen = torch.Generator(device="cuda").manual_seed(13)
    weights = (torch.randn(w.nnz, generator=gen, device="cuda") * w.w_std).to(t_in)
    packed = torch.zeros(rb.rbgp_packed_bytes(mask, dtype), dtype=torch.uint8, device="cuda")
    rb.rbgp_pack_device(mask, dtype, weights.data_ptr(), packed.data_ptr())
    out = torch.full((w.M + 1, N), -77.0, device="cuda")
    if side:
        images, C = N // side ** 2, w.K // 9
        X = torch.zeros((C, images, side + 2, side + 2), dtype=t_in, device="cuda")
        X[:, :, 1:-1, 1:-1] = torch.randn((C, images, side, side), generator=gen, device="cuda")
        rb.rbgp_conv3x3(mask, dtype, w.M, C, images, side, side, packed.data_ptr(), X.data_ptr(), out.data_ptr(), N)
        I = torch.stack([X[:, :, dy:dy + side, dx:dx + side] for dy in range(3) for dx in range(3)], 1).reshape(w.K, N).double()
    else:
        ldI = -(-N // 8) * 8
        rows = torch.randn((w.K, ldI), generator=gen, device="cuda").to(t_in)
        rb.rbgp_spmm(mask, dtype, w.M, w.K, N, packed.data_ptr(), rows.data_ptr(), ldI, out.data_ptr(), N)
        I = rows[:, :N].double()
    torch.cuda.synchronize()
    assert (out[w.M] == -77).all()
    cols = torch.from_numpy(rb.rbgp_mask_columns(mask).reshape(w.M, -1).astype("int64")).cuda()
    dense = torch.zeros((w.M, w.K), dtype=torch.float64, device="cuda").scatter_(1, cols, weights.view(w.M, -1).double())
    bound = cols.shape[1] * 2.0 ** -24 * (dense.abs() @ I.abs())   # (one fp32 rounding per product and sum, in any order)
    assert bool(((out[:w.M].double() - dense @ I).abs() <= bound).all())
