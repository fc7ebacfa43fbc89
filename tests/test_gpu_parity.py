"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle
on the same seeded inputs, element by element."""
from dataclasses import replace

import numpy as np
import pytest

from oracle import rbgp_oracle as orc
from paper_2006_13486_amd import binding as rb
from paper_2006_13486_amd import workloads as wl
from tests import gpu_harness as gh

pytestmark = pytest.mark.gpu

GEN, MFMA, REG = rb.KERNEL_GENERIC, rb.KERNEL_MFMA, rb.KERNEL_MFMA_REG
FILLED = rb.KERNEL_MFMA_REG_FILLED


# ------------------------------------------------------------------ fixed configurations, full size
@pytest.mark.parametrize("w", wl.CONFIGS, ids=lambda w: w.name)
def test_config_full_size_default_launch(w):
    """The launch configuration bench.py times (library defaults)."""
    gh.check_parity(w, expect_kernel=REG)


@pytest.mark.parametrize("w", [wl.TINY, wl.VGG19_CONV5, wl.VGG19_CONV3_BF16], ids=lambda w: w.name)
def test_config_generic_kernel(w):
    gh.check_parity(w, N=min(w.N, 1024), kernel=GEN, expect_kernel=GEN)


@pytest.mark.parametrize("tune", [(1, 64, 0), (2, 128, 0), (1, 64, 2), (2, 128, 1)])
@pytest.mark.parametrize("w", [wl.VGG19_CONV5, wl.VGG19_CONV3_BF16, wl.WRN_G1], ids=lambda w: w.name)
def test_config_tile_shapes(w, tune):
    gh.check_parity(w, N=1536 if w.N > 4096 else w.N, kernel=MFMA, tune=tune)


@pytest.mark.parametrize("pairing", [0, 1, 2])
@pytest.mark.parametrize("w", [wl.TINY, wl.VGG19_CONV5, wl.VGG19_CONV3_BF16, wl.WRN_G1], ids=lambda w: w.name)
def test_config_register_family_row_pairing(w, pairing):
    """Fixed pairs of tile rows (1) and tile-by-tile pairing (2; fp32 masks with two tile rows of 8
    per MFMA group only: the conv5 shape, the others must refuse it), at a ragged N."""
    N = 1000 if w.N > 4096 else w.N
    if pairing == 2 and w is not wl.VGG19_CONV5:
        with pytest.raises(rb.RbgpError) as e:
            gh.check_parity(w, N=N, kernel=REG, tune=(0, 0, 0, pairing), expect_kernel=REG)
        assert e.value.code == rb.EUNSUPPORTED
        return
    gh.check_parity(w, N=N, kernel=REG, tune=(0, 0, 0, pairing), expect_kernel=REG)


# masks with two tile rows of 8 rows per MFMA group, for the tile-by-tile pairing of the fp32 register kernels
PAIRING_SHAPES = [
    ((4, 4, 4, 2), (4, 4, 8, 9), (2, 4, 2, 9)),     # 4 tile rows: one quad
    ((8, 2, 2, 3), (8, 2, 4, 3), (4, 2, 2, 3)),     # R = 6 (two idle rows per half), stages of 12 steps padded to 18
    ((6, 4, 2, 2), (4, 1, 4, 9), (2, 1, 2, 9)),     # 6 tile rows: a quad with two rows missing
    ((2, 8, 2, 1), (4, 2, 2, 4), (2, 2, 1, 4)),     # 2 tile rows: a quad with one L row and one H row
    ((16, 1, 2, 8), (16, 2, 4, 2), (4, 2, 2, 2)),   # 16 tile rows of degree 4 (two lifts): tiles without a partner
    ((4, 21, 2, 1), (4, 1, 2, 9), (2, 1, 1, 9)),    # |G_r.U| = 21: three tile rows of 7 per row of G_o
]


@pytest.mark.parametrize("shape", range(len(PAIRING_SHAPES)))
def test_fp32_register_family_tile_by_tile_pairing(shape):
    """The pairing kernel against the oracle (and the fixed-pair kernel on the same inputs) on small masks
    that exercise incomplete quads, idle rows, padded stages and partnerless tiles, at two ragged N with
    an odd leading dimension; the host tables pass the library's own consistency check."""
    a, c, d = PAIRING_SHAPES[shape]
    for N in (200, 129):
        w = wl.Workload(f"pairing_{shape}", a, c, d, N, wl.F32, 100 + shape, 200 + shape, 300 + shape, 1.0)
        rb.rbgp_mask_check_tables(gh.make_mask(w))
        assert rb.rbgp_mask_reg_plan(gh.make_mask(w))[7] > 0
        gh.check_parity(w, kernel=REG, tune=(0, 0, 0, 2), ld_pad=3, expect_kernel=REG)
        gh.check_parity(w, kernel=REG, tune=(0, 0, 0, 1), ld_pad=3, expect_kernel=REG)


@pytest.mark.parametrize("cw", [64, 128])
@pytest.mark.parametrize("split", [1, 2, 4])
@pytest.mark.parametrize("groups", [1, 2, 4])
def test_bf16_register_family_row_groups_and_stage_split(groups, split, cw):
    """bf16 register kernels: every (16-row groups per wave, waves per column tile,
    columns per wave) combination, on the conv3 shape (ragged last tile) and on shapes
    with fewer tile rows than one cluster holds, a partial 4-row block, an odd stage
    count, 12 tile rows."""
    tune = (0, cw, 0, 0, groups, split)
    gh.check_parity(wl.VGG19_CONV3_BF16, N=1000, kernel=REG, tune=tune, expect_kernel=REG)
    w = wl.Workload("bf16_small_cluster", (2, 1, 4, 3), (4, 2, 4, 9), (2, 2, 2, 9), 330, wl.BF16, 11, 12, 13, 1.0)
    gh.check_parity(w, kernel=REG, tune=tune, ld_pad=6, expect_kernel=REG)   # (ldI must be a multiple of 8)
    w = wl.Workload("bf16_rs4", (6, 2, 4, 2), (6, 1, 4, 9), (3, 1, 2, 9), 200, wl.BF16, 21, 22, 23, 1.0)
    gh.check_parity(w, kernel=REG, tune=tune, expect_kernel=REG)
    w = wl.Workload("bf16_12_tile_rows", (12, 1, 2, 3), (8, 1, 4, 9), (2, 1, 2, 9), 136, wl.BF16, 31, 32, 33, 1.0)
    gh.check_parity(w, kernel=REG, tune=tune, expect_kernel=REG)


@pytest.mark.parametrize("split", [2, 4])
def test_fp32_register_family_stage_split(split):
    """fp32 register kernels with the stage list split over 2 or 4 waves (LDS reduction)."""
    tune = (0, 0, 0, 0, 0, split)
    for w, N in [(wl.TINY, None), (wl.VGG19_CONV5, 520), (wl.WRN_G1, 1000)]:
        gh.check_parity(w, N=N, kernel=REG, tune=tune, expect_kernel=REG)
    w = wl.Workload("fp32_small_cluster", (2, 1, 4, 3), (4, 2, 4, 9), (2, 2, 2, 9), 331, wl.F32, 11, 12, 13, 1.0)
    gh.check_parity(w, kernel=REG, tune=tune, ld_pad=2, expect_kernel=REG)   # odd leading dimension
    gh.check_parity(wl.VGG19_CONV5, kernel=REG, tune=tune, expect_kernel=REG)


def test_bf16_register_family_full_size_split_shapes():
    for tune in [(0, 128, 0, 0, 4, 4), (0, 128, 0, 0, 2, 2), (0, 64, 0, 0, 4, 2), (0, 64, 0, 0, 2, 2), (0, 64, 0, 0, 1, 1)]:
        gh.check_parity(wl.VGG19_CONV3_BF16, kernel=REG, tune=tune, expect_kernel=REG)


def test_lds_family_full_size():
    for w in (wl.VGG19_CONV5, wl.VGG19_CONV3_BF16, wl.WRN_G1):
        gh.check_parity(w, kernel=MFMA, expect_kernel=MFMA)


# ------------------------------------------------------------------ ragged and degenerate sizes
@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("N,ld_pad", [(1, 7), (63, 1), (64, 0), (65, 3), (200, 8), (257, 15)])
def test_ragged_columns(N, ld_pad, dtype):
    """Column counts that leave a partial tile, with a padded leading dimension
    (pad columns of O must stay untouched)."""
    epc = 8 if dtype == wl.BF16 else 4
    pad = (-N) % epc + ld_pad // epc * epc            # keeps ldI a multiple of the 16-byte chunk
    w = replace(wl.VGG19_CONV5, rows=(4, 4, 4, 2), cols=(4, 4, 8, 9), row_deg=(2, 4, 2, 9), dtype=dtype,
                name=f"ragged_{dtype}")
    for tune in [(1, 64, 0), (2, 128, 0)]:
        gh.check_parity(w, N=N, kernel=MFMA, tune=tune, ld_pad=pad)
    gh.check_parity(w, N=N, kernel=GEN, ld_pad=ld_pad)
    for pairing in (1, 2):
        gh.check_parity(w, N=N, kernel=REG, tune=(0, 0, 0, pairing if dtype == wl.F32 else 1), ld_pad=ld_pad if dtype == wl.F32 else pad,
                        expect_kernel=REG)
    if dtype == wl.BF16:                              # 128-column wave tiles, with and without a stage split
        gh.check_parity(w, N=N, kernel=REG, tune=(0, 128), ld_pad=pad, expect_kernel=REG)
        gh.check_parity(w, N=N, kernel=REG, tune=(0, 128, 0, 0, 2, 2), ld_pad=pad, expect_kernel=REG)


def test_empty_input_is_a_noop():
    import torch
    w = wl.TINY
    mask = rb.rbgp_make_mask(w.rows, w.cols, w.row_deg, 1)
    O = torch.full((w.M, 4), 5.0, device="cuda:0")
    rb.rbgp_spmm(mask, w.dtype, w.M, w.K, 0, 0, 0, 0, O.data_ptr(), 0, 0)
    torch.cuda.synchronize()
    assert bool((O == 5.0).all())


def test_misaligned_input_is_rejected_by_the_mfma_family():
    import torch
    w = wl.TINY
    mask = rb.rbgp_make_mask(w.rows, w.cols, w.row_deg, 1)
    rb.rbgp_mask_set_kernel(mask, MFMA)
    packed = torch.zeros(rb.rbgp_packed_bytes(mask, w.dtype), dtype=torch.uint8, device="cuda:0")
    I = torch.zeros(w.K * 70 + 8, device="cuda:0")
    O = torch.zeros(w.M * 70, device="cuda:0")
    with pytest.raises(rb.RbgpError) as ei:
        rb.rbgp_spmm(mask, w.dtype, w.M, w.K, 66, packed.data_ptr(), I.data_ptr(), 66, O.data_ptr(), 66, 0)
    assert ei.value.code == rb.ESHAPE
    with pytest.raises(rb.RbgpError) as ei:
        rb.rbgp_spmm(mask, w.dtype, w.M, w.K, 64, packed.data_ptr(), I.data_ptr() + 4, 64, O.data_ptr(), 64, 0)
    assert ei.value.code == rb.ESHAPE
    torch.cuda.synchronize()


# ------------------------------------------------------------------ exact cases
@pytest.mark.parametrize("kernel", [GEN, MFMA, REG])
@pytest.mark.parametrize("w", [wl.TINY, replace(wl.WRN_G1, N=576)], ids=lambda w: w.name)
def test_one_hot_input_returns_dense_weights_exactly(w, kernel):
    """I = identity: every output is one kept weight times 1 plus zeros, exact
    in fp32.  Pins the pack permutation and every index bit for bit."""
    vals = wl.kept_weights(w)
    I = np.eye(w.K, dtype=np.float32)
    out, _ = gh.library_spmm(w, vals, I, kernel, tag="one-hot")
    Bs, _ = orc.sample_factors(w.rows, w.cols, w.row_deg, w.mask_seed)
    W = orc.scatter_values(orc.kron_mask(Bs), vals)
    assert np.array_equal(out, W)


def test_one_hot_bf16_exact():
    w = replace(wl.TINY, dtype=wl.BF16, name="tiny_bf16")
    vb = wl.to_bf16_bits(wl.kept_weights(w))
    Ib = wl.to_bf16_bits(np.eye(w.K, dtype=np.float32))
    for kernel in (GEN, MFMA, REG):
        out, _ = gh.library_spmm(w, vb, Ib, kernel, tag="one-hot bf16")
        Bs, _ = orc.sample_factors(w.rows, w.cols, w.row_deg, w.mask_seed)
        W = orc.scatter_values(orc.kron_mask(Bs), wl.bf16_bits_as_f32(vb))
        assert np.array_equal(out, W)


def test_all_complete_factors_is_a_dense_gemm():
    w = wl.Workload("dense_32x72", (2, 4, 2, 2), (1, 2, 4, 9), (1, 2, 4, 9), 300, wl.F32, 1, 2, 3)
    if gh.family_covers(w, MFMA):      # (a complete G_i counts as row repetition: 16 rows share a column set here,
        gh.check_parity(w, kernel=MFMA, ld_pad=0)   #  more than the LDS family's blocks hold)
    gh.check_parity(w, kernel=REG, expect_kernel=REG)
    gh.check_parity(w, kernel=GEN)


# ------------------------------------------------------------------ shapes across the kernel table
FUZZ = [
    # rows, cols, row_deg  (G_r, G_b complete)                     covers
    ((2, 1, 2, 1), (4, 1, 4, 1), (2, 1, 2, 1)),                    # R=1, KS=2
    ((4, 2, 8, 1), (4, 3, 8, 1), (2, 3, 4, 1)),                    # R=2, KS=4, |G_r.V|=3
    ((2, 1, 16, 4), (2, 1, 16, 2), (2, 1, 8, 2)),                  # R=4, KS=16
    ((4, 4, 16, 1), (8, 1, 32, 1), (4, 1, 8, 1)),                  # Table-2-like: R=4, KS=8, 16 groups
    ((2, 2, 32, 2), (4, 1, 64, 1), (2, 1, 32, 1)),                 # KS=32, 32 groups
    ((4, 2, 4, 4), (4, 2, 8, 9), (2, 2, 4, 9)),                    # R=8, KS=36
    ((2, 4, 4, 2), (2, 2, 16, 9), (1, 2, 8, 9)),                   # KS=72
    ((4, 1, 4, 3), (4, 2, 4, 9), (2, 2, 2, 9)),                    # R=3 (partial 4-row block)
    ((2, 3, 4, 2), (2, 2, 4, 9), (1, 2, 2, 9)),                    # R=6 (one full, one partial block)
    # the remaining (stage size, row group) pairs of the register family's kernel table
    ((2, 4, 16, 1), (2, 1, 16, 1), (2, 1, 8, 1)),                  # KC=8,  RS=4
    ((4, 2, 4, 1), (4, 1, 4, 9), (2, 1, 2, 9)),                    # KC=18, RS=2
    ((4, 2, 4, 1), (4, 2, 4, 9), (2, 2, 2, 9)),                    # KC=36, RS=2
    ((4, 1, 4, 2), (4, 2, 8, 9), (2, 2, 4, 9)),                    # KC=72, RS=2
    ((4, 2, 4, 2), (4, 1, 4, 9), (2, 1, 2, 9)),                    # KC=18, RS=4
    ((4, 2, 4, 2), (4, 2, 8, 9), (2, 2, 4, 9)),                    # KC=72, RS=4
    ((4, 4, 4, 2), (4, 1, 4, 9), (2, 1, 2, 9)),                    # KC=18, RS=8
    # stages whose length is padded to the next kernel size
    ((4, 2, 4, 2), (4, 2, 4, 3), (2, 2, 2, 3)),                    # 12 steps in KC=18
    ((2, 1, 8, 4), (2, 3, 8, 3), (1, 3, 2, 3)),                    # 18 = 3 x 2 x 3
    ((4, 2, 4, 1), (4, 1, 12, 9), (2, 1, 6, 9)),                   # 54 steps in KC=72
    ((4, 4, 4, 1), (4, 5, 4, 1), (2, 5, 1, 1)),                    # 5 steps in KC=8
    ((4, 1, 8, 3), (4, 3, 8, 3), (2, 3, 2, 3)),                    # R=3, 18 steps
    # more than 16 rows per tile row: rows of G_r move into the tile-row index
    ((2, 8, 4, 3), (2, 2, 4, 9), (1, 2, 2, 9)),                    # R=24 -> 2 x 12
    ((4, 4, 2, 9), (4, 4, 4, 2), (2, 4, 2, 2)),                    # R=36 -> 4 x 9 (a transposed 3x3 layer)
    # a complete G_i joins G_r in the kernels' view (all the sparsity in G_o)
    ((2, 2, 32, 2), (4, 1, 32, 1), (2, 1, 32, 1)),                 # 128 rows share a column set
    ((2, 4, 4, 2), (2, 2, 8, 9), (1, 2, 8, 9)),                    # R=32 -> 2 x 16, stages of 72
    ((8, 4, 4, 2), (8, 4, 8, 9), (4, 4, 8, 9)),                    # a VGG19 layer at density 1/2
    ((4, 2, 2, 4), (4, 2, 4, 9), (2, 2, 4, 9)),                    # R=16, stages of 36
]
REG_COVERED = set(range(5, 23))               # must run on the register family


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("idx", range(len(FUZZ)))
def test_shapes_across_the_kernel_table(idx, dtype):
    rows, cols, deg = FUZZ[idx]
    w = wl.Workload(f"fuzz{idx}_{dtype}", rows, cols, deg, 328, dtype, 100 + idx, 200 + idx, 300 + idx, 1.0)
    if gh.family_covers(w, MFMA):
        gh.check_parity(w, kernel=MFMA, tune=(1, 64, 0))
        gh.check_parity(w, kernel=MFMA, tune=(2, 128, 0))
    else:
        assert idx >= 9                       # the first nine shapes are inside the LDS family's table
    gh.check_parity(w, kernel=GEN)
    if gh.family_covers(w, FILLED):           # few rows per column set and a sparse G_i: the mask with G_i filled in
        gh.check_parity(w, kernel=FILLED, expect_kernel=FILLED)
        gh.check_parity(w, kernel=FILLED, tune=(0, 0, 0, 0, 0, 2), ld_pad=8, expect_kernel=FILLED)
    covered = gh.family_covers(w, REG)
    assert covered or idx not in REG_COVERED
    if covered:
        # tile-by-tile pairing of the tile rows where the library's plan has it (fp32, two tile rows per MFMA group)
        pairing = dtype == wl.F32 and rb.rbgp_mask_reg_plan(gh.make_mask(w))[7] > 0
        for tune in [(0, 0, 0, 1), (0, 0, 0, 0, 0, 2)] + ([(0, 0, 0, 2)] if pairing else []) + \
                ([(0, 64, 0, 0, 2, 1), (0, 128, 0, 0, 1, 4)] if dtype == wl.BF16 else []):
            gh.check_parity(w, kernel=REG, tune=tune, expect_kernel=REG)


# stage lists as long as or longer than the 64 stages one wave holds: split over 2 or 4 waves of the workgroup
LONG_LISTS = [
    ((4, 2, 2, 1), (128, 1, 2, 1), (64, 1, 2, 1)),     # 64 tiles per tile row (complete G_i joins G_r): 2 waves
    ((4, 4, 1, 2), (256, 1, 1, 2), (128, 1, 1, 2)),    # G_o of 256 tile columns at 1/2, two tile rows per cluster: 3 waves
    ((4, 2, 4, 2), (64, 4, 8, 9), (32, 4, 4, 9)),      # two stages of 72 steps per tile, four tile rows per cluster
    ((8, 1, 4, 1), (64, 2, 4, 2), (16, 2, 1, 2)),      # clusters of 8 tile rows whose union fills one wave's table to the last lane
]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("idx", range(len(LONG_LISTS)))
def test_register_family_stage_lists_beyond_one_wave(idx, dtype):
    """Clusters that walk 64..256 stages: beyond 64 the register kernels split the list over the waves of a workgroup
    whatever N is (default launch), also with the largest split asked for; the tables pass the self check."""
    rows, cols, deg = LONG_LISTS[idx]
    for N in (200, 1100):
        w = wl.Workload(f"long{idx}_{dtype}", rows, cols, deg, N, dtype, 400 + idx, 500 + idx, 600 + idx, 1.0)
        m = gh.make_mask(w)
        rb.rbgp_mask_check_tables(m)
        assert 64 <= rb.rbgp_mask_reg_plan(m)[5] <= 256
        gh.check_parity(w, kernel=REG, expect_kernel=REG, ld_pad=8)
        gh.check_parity(w, kernel=REG, tune=(0, 0, 0, 0, 0, 4), expect_kernel=REG)
    if rb.rbgp_mask_reg_plan(m)[5] > 64:         # one wave cannot hold this list
        with pytest.raises(rb.RbgpError) as e:
            gh.check_parity(w, kernel=REG, tune=(0, 0, 0, 0, 0, 1), expect_kernel=REG)
        assert e.value.code == rb.EUNSUPPORTED
    else:
        gh.check_parity(w, kernel=REG, tune=(0, 0, 0, 0, 0, 1), expect_kernel=REG)


# masks with at most four rows per column set and a sparse G_i (the shapes of Table 3's slow rows, small)
FILLED_SHAPES = [
    ((4, 1, 16, 1), (8, 1, 8, 1), (4, 1, 4, 1)),       # R = 1: 16 rows per tile row after the fill, stages of 8 steps
    ((2, 2, 32, 1), (4, 1, 32, 1), (2, 1, 8, 1)),      # R = 2, G_i at 1/4: 64 rows -> four 16-row groups per tile row
    ((4, 1, 8, 4), (8, 3, 8, 2), (2, 3, 2, 2)),        # R = 4 from G_b, |G_r.V| = 3: stages of 48 steps padded to 72
    ((2, 1, 12, 1), (64, 1, 4, 1), (64, 1, 2, 1)),     # complete G_o of 64 tiles: a stage list split over two waves
    ((8, 1, 4, 3), (8, 1, 8, 1), (2, 1, 2, 1)),        # R = 3, 12 rows per tile row: a partial 16-row group
]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("idx", range(len(FILLED_SHAPES)))
def test_register_family_on_the_mask_with_g_i_filled_in(idx, dtype):
    """RBGP_KERNEL_MFMA_REG_FILLED against the oracle of the ORIGINAL mask: the zeros stored where G_i has no
    edge must change nothing; forward and transposed products, ragged N, padded leading dimension."""
    rows, cols, deg = FILLED_SHAPES[idx]
    w = wl.Workload(f"filled{idx}_{dtype}", rows, cols, deg, 328, dtype, 700 + idx, 800 + idx, 900 + idx, 1.0)   # (bf16: ldI % 8 == 0)
    m = gh.make_mask(w)
    rb.rbgp_mask_check_tables(m)
    assert rb.rbgp_mask_reg_plan(m)[13] > 0
    gh.check_parity(w, kernel=FILLED, expect_kernel=FILLED)
    gh.check_parity(w, N=1096, kernel=FILLED, ld_pad=8, expect_kernel=FILLED)
    # transposed product: the filled family where the transposed mask has one, else whatever it runs on
    (vl, Il, dOl), f32 = gh.backward_inputs(w)
    want_dI, den, _, _ = gh.oracle_backward(w, *f32)
    mt = rb.rbgp_mask_transpose(m)
    kernel = FILLED if rb.rbgp_mask_reg_plan(mt)[13] > 0 else rb.KERNEL_AUTO
    got, used = gh.library_spmm_transposed(w, vl, dOl, kernel=kernel)
    assert kernel == rb.KERNEL_AUTO or used == FILLED
    assert orc.normalised_error(got, want_dI, den) <= gh.TOL[w.dtype]


def test_filled_family_is_what_auto_takes_for_one_row_per_column_set():
    """Table 3, G_r = G_b = (1, 1): the default launch is the filled family (both dtypes); never for the mask of a
    lowered 3x3 convolution, never where no filled mask exists."""
    w = wl.sdmm4096_table3(1, 1, 3)
    m = gh.make_mask(w)
    assert rb.rbgp_mask_kernel(m, wl.F32) == FILLED and rb.rbgp_mask_kernel(m, wl.BF16) == FILLED
    assert rb.rbgp_mask_kernel(gh.make_mask(wl.WRN_G1), wl.F32) == REG
    with pytest.raises(rb.RbgpError) as e:
        rb.rbgp_mask_set_kernel(gh.make_mask(wl.VGG19_CONV5), FILLED)
    assert e.value.code == rb.EUNSUPPORTED


# masks whose rows of G_r move into the tile-row index (more than 16 rows per column set): fp32 waves that take 2 or 4
# of the tile rows that share their tiles
ROW_GROUP_SHAPES = [
    ((2, 8, 4, 3), (2, 2, 4, 9), (1, 2, 2, 9), (2,)),        # R = 24 -> 2 x 12, stages of 36
    ((4, 4, 2, 11), (4, 4, 4, 2), (2, 4, 2, 2), (2, 4)),     # R = 44 -> 4 x 11, stages of 16 in 18
    ((2, 2, 32, 2), (4, 1, 32, 1), (2, 1, 32, 1), (2,)),     # complete G_i: 128 rows -> 8 x 16, stages of 32 (no kernel of 4 groups)
    ((2, 4, 4, 2), (2, 2, 8, 9), (1, 2, 8, 9), (2,)),        # R = 32 -> 2 x 16, stages of 72
    ((4, 8, 1, 8), (8, 2, 1, 9), (4, 2, 1, 9), (2, 4)),      # R = 64 -> 4 x 16, stages of 18
]


@pytest.mark.parametrize("idx", range(len(ROW_GROUP_SHAPES)))
def test_fp32_register_family_row_groups_per_wave(idx):
    """RBGP_TUNE_ROW_GROUPS on the fp32 register kernels (2 or 4 tile rows with the same tiles per wave), ragged N,
    padded leading dimension, alone and with a split stage list; refused where the tile rows do not come in such groups."""
    rows, cols, deg, groups = ROW_GROUP_SHAPES[idx]
    w = wl.Workload(f"rowgroups{idx}", rows, cols, deg, 333, wl.F32, 40 + idx, 50 + idx, 60 + idx, 1.0)
    for ng in groups:
        gh.check_parity(w, kernel=REG, tune=(0, 0, 0, 0, ng), ld_pad=3, expect_kernel=REG)
        gh.check_parity(w, N=64, kernel=REG, tune=(0, 0, 0, 0, ng), expect_kernel=REG)
    gh.check_parity(w, kernel=REG, tune=(0, 0, 0, 0, 2, 2), expect_kernel=REG)     # with a split stage list as well
    gh.check_parity(w, kernel=REG, tune=(0, 0, 0, 0, 2, 0, 0, 2), ld_pad=1, expect_kernel=REG)   # two register sets
    gh.check_parity(w, N=200, kernel=REG, tune=(0, 0, 0, 0, groups[-1], 4), ld_pad=1, expect_kernel=REG)
    if 4 not in groups:
        with pytest.raises(rb.RbgpError) as e:
            gh.check_parity(w, kernel=REG, tune=(0, 0, 0, 0, 4), expect_kernel=REG)
        assert e.value.code == rb.EUNSUPPORTED


# masks whose tile rows come in groups of 2 or 8 with the same tiles, with stages of 8 to 72 steps (whole and partial
# blocks of 16, groups of 16 and of fewer rows); the last two runs: lists of one stage, and of 96 (split over waves)
SPLIT_OPERAND_SHAPES = [
    ((4, 32, 1, 1), (4, 8, 4, 1), (2, 8, 4, 1), 2),
    ((4, 32, 2, 4), (4, 2, 8, 9), (2, 2, 4, 9), 8),
    ((2, 16, 2, 9), (4, 2, 4, 9), (2, 2, 2, 9), 8),
    ((2, 8, 1, 16), (2, 4, 16, 1), (1, 4, 16, 1), 8),
    ((4, 64, 2, 2), (4, 2, 4, 2), (2, 2, 2, 2), 8),
    ((2, 128, 2, 1), (4, 3, 4, 2), (2, 3, 2, 2), 8),
    ((4, 32, 1, 1), (192, 1, 16, 1), (96, 1, 16, 1), 2),
]


@pytest.mark.parametrize("idx", range(len(SPLIT_OPERAND_SHAPES)))
def test_fp32_register_family_split_operands(idx):
    """RBGP_TUNE_SPLIT_OPERANDS: fp32 products on the bf16 matrix core, waves by themselves and four sharing their
    columns; widths around the 128-column tile, padded leading dimensions, split stage lists."""
    rows, cols, deg, group = SPLIT_OPERAND_SHAPES[idx]
    w = wl.Workload(f"split{idx}", rows, cols, deg, 333, wl.F32, 140 + idx, 150 + idx, 160 + idx, 1.0)
    for N, pad in ((1, 0), (97, 3), (128, 0), (129, 5), (400, 4)):
        gh.check_parity(w, N=N, kernel=REG, tune=(0,) * 8 + (2,), ld_pad=pad, expect_kernel=REG)
        if group == 8:
            gh.check_parity(w, N=N, kernel=REG, tune=(0,) * 8 + (3,), ld_pad=pad, expect_kernel=REG)
    for s in (2, 4):
        gh.check_parity(w, N=200, kernel=REG, tune=(0, 0, 0, 0, 0, s, 0, 0, 2), ld_pad=1, expect_kernel=REG)
    for tune in (((0,) * 8 + (3,)) if group != 8 else (0, 0, 0, 0, 0, 2, 0, 0, 3), (0, 0, 0, 0, 2, 0, 0, 0, 2)):
        with pytest.raises(rb.RbgpError) as e:
            gh.check_parity(w, kernel=REG, tune=tune, expect_kernel=REG)
        assert e.value.code == rb.EUNSUPPORTED


@pytest.mark.parametrize("variant", [2, 3])
def test_split_operands_keep_infinities_and_other_columns(variant):
    """An operand that is infinite, not a number, or beyond the largest bf16 number: sums that the fp32 kernel gives as
    finite or infinite come out the same, columns without such operands keep every bit; tiny operands lose nothing."""
    w = wl.Workload("split_inf", (2, 128, 1, 1), (4, 2, 16, 1), (2, 2, 16, 1), 333, wl.F32, 1, 2, 3, 1.0)
    N = 200
    vl, Il, vf, If = gh.host_inputs(w, N)
    run = lambda X, v: gh.library_spmm(w, vl, X, kernel=REG, tune=(0,) * 8 + (v,), tag="split operands")[0]
    clean = run(Il, variant)
    bad = Il.copy()
    bad[3, 5], bad[7, 60], bad[40, 130], bad[41, 131] = np.inf, np.nan, -np.inf, np.float32(3.4e38)
    got, ref = run(bad, variant), run(bad, 1)
    cols = [5, 60, 130, 131]
    others = np.ones(N, bool)
    others[cols] = False
    assert np.array_equal(got[:, others].view(np.uint32), clean[:, others].view(np.uint32))
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
    both = np.isfinite(ref[:, 131])
    assert np.allclose(got[both, 131], ref[both, 131], rtol=1e-5)
    for scale in (2.0 ** -60, 2.0 ** 60):   # (a power of two only moves the exponent)
        assert np.array_equal(run(Il * np.float32(scale), variant), clean * np.float32(scale))
    tiny = np.ones((1, N), np.float32)      # (columns whose bf16 parts would be denormal; a power of two again)
    tiny[:, 100:140] = 2.0 ** -120
    got, ref = run(Il * tiny, variant), run(Il, 1)
    assert np.array_equal(got[:, :100].view(np.uint32), clean[:, :100].view(np.uint32))
    small = got[:, 100:140].astype(np.float64) * 2.0 ** 120
    bound = 1e-6 * np.abs(ref[:, 100:140]).max(axis=0)      # (64 products each: a few rounding errors of 6e-8)
    assert (np.abs(small - ref[:, 100:140]) <= bound).all()


@pytest.mark.parametrize("kernel,variant", [(REG, 1), (REG, 2), (REG, 3), (MFMA, 1), (MFMA, 2)])
def test_split_operands_keep_the_bits_of_tiny_operands(kernel, variant):
    """Rows of W and columns of I down to fp32's denormals among ordinary and huge ones, so that one lane holds sums of
    very different sizes and tiny weights meet huge activations: every sum by itself is an fp32 sum of its n products,
    within n + 8 roundings of the products' size (8: the operands' parts that are left out) and of denormals."""
    shape = ((2, 128, 1, 1), (4, 2, 16, 1), (2, 2, 16, 1)) if kernel == REG else ((4, 4, 32, 1), (8, 1, 32, 1), (4, 1, 8, 1))
    w = wl.Workload("split_tiny", *shape, 333, wl.F32, 21, 22, 23, 1.0)
    N, rng = 200, np.random.default_rng(24)
    vals, I = wl.kept_weights(w).reshape(w.M, w.rowdeg), wl.activations(w, N)
    vals = vals * rng.choice(2.0 ** np.array([0, 0, 0, 8, -40, -100, -112, -118, -124, -130]), (w.M, 1)).astype(np.float32)
    I = I * rng.choice(2.0 ** np.array([0, 0, 0, 60, -20, -60, -90, -118, -126, -135]), (1, N)).astype(np.float32)
    out, used = gh.library_spmm(w, vals, I, kernel=kernel, tune=(0,) * 8 + (variant,), tag="tiny operands")
    assert used == kernel
    mask = rb.rbgp_mask_dense(gh.make_mask(w)).reshape(w.M, w.K).astype(bool)
    W = np.zeros((w.M, w.K))
    W[mask] = vals.reshape(-1)
    X, n = I.astype(np.float64), w.rowdeg
    bound = (n + 8) * (2.0 ** -24 * (np.abs(W) @ np.abs(X)) + 2.0 ** -150)
    assert (np.abs(out - W @ X) <= bound).all()


@pytest.mark.parametrize("out_bf16", [False, True])
@pytest.mark.parametrize("idx", [0, 3, 5, 6])
def test_bf16_register_family_shared_columns(idx, out_bf16):
    """RBGP_TUNE_SHARED_COLUMNS: bf16 workgroups that pass I through LDS, every arrangement of their waves; widths around
    the 128-column tiles and the workgroups' widths, lists of one stage; the sums are those of one wave per list."""
    rows, cols, deg, group = SPLIT_OPERAND_SHAPES[idx]
    w = wl.Workload(f"shared{idx}", rows, cols, deg, 333, wl.BF16, 170 + idx, 180 + idx, 190 + idx, 1.0)
    for N, pad in ((1, 7), (128, 0), (131, 5), (520, 8)):
        vl, Il, vf, If = gh.host_inputs(w, N)
        ref, den = gh.oracle_spmm(w, vf, If)
        for value, need in ((2, 2), (3, 4), (4, 8), (5, 4), (6, 8)):
            tune = (0,) * 9 + (value,)
            if need > group or idx == 6:      # (the last shape: lists of more than 64 stages)
                with pytest.raises(rb.RbgpError) as e:
                    gh.library_spmm(w, vl, Il, kernel=REG, tune=tune, ld_pad=pad)
                assert e.value.code == rb.EUNSUPPORTED
                continue
            out, used = gh.library_spmm(w, vl, Il, kernel=REG, tune=tune, ld_pad=pad, out_bf16=out_bf16)
            assert used == REG
            full = out if not out_bf16 else gh.library_spmm(w, vl, Il, kernel=REG, tune=tune, ld_pad=pad)[0]
            assert orc.normalised_error(full, ref, den) <= 4e-6      # (bf16 products are exact in fp32)
            if out_bf16:
                assert np.array_equal(out, wl.bf16_bits_as_f32(wl.to_bf16_bits(full)))


# masks whose merged tile columns are walked in stages of 64 steps, in the packed layout of 72: one stage, four, sixteen
STAGES_OF_64 = [((8, 2, 2, 2), (8, 1, 4, 4), (8, 1, 2, 4)), ((8, 2, 2, 2), (32, 1, 4, 4), (32, 1, 2, 4)),
                ((8, 4, 2, 2), (64, 2, 4, 4), (64, 2, 2, 4))]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("idx", range(len(STAGES_OF_64)))
def test_stages_of_64_steps_in_the_layout_of_72(idx, dtype):
    """Every kernel that leaves out the padding of these stages (its weight fragments and row tables are those of 72
    steps): bf16 on 64 and 128 columns, one and two row groups, one and two register sets; fp32 with one and two row
    groups; whole and split lists, odd widths, padded rows."""
    rows, cols, deg = STAGES_OF_64[idx]
    w = wl.Workload(f"stages64_{idx}", rows, cols, deg, 131, dtype, 51 + idx, 52, 53, 1.0)
    assert rb.rbgp_mask_reg_plan(gh.make_mask(w))[14] == 16      # (merged: whole groups of 16 rows)
    ks = (0, 2) if idx else (0,)
    if dtype == wl.F32:
        tunes = [(0, 0, 0, 0, g, s, 0, rs, 1, 0) for g, rs in ((1, 1), (1, 2), (2, 0)) for s in ks]
    else:
        tunes = [(0, c, 0, 0, g, s, 0, rs, 0, 1) for c, rs in ((64, 0), (128, 1), (128, 2)) for g in (1, 2) for s in ks]
    for N, pad in ((1, 7), (131, 5), (328, 8)):
        vl, Il, vf, If = gh.host_inputs(w, N)
        ref, den = gh.oracle_spmm(w, vf, If)
        for tune in tunes:
            out, used = gh.library_spmm(w, vl, Il, kernel=REG, tune=tune, ld_pad=pad, tag="stages of 64")
            assert used == REG
            assert orc.normalised_error(out, ref, den) <= 4e-6


# many rows per tile, two of four columns of G_i kept: 96 and 120 rows (the last group of 32 in part), nine tile rows per
# row of G_o, lists of one, four, eight and twelve stages
MANY_ROWS = [((4, 4, 8, 3), (8, 4, 4, 2), (4, 4, 2, 2)), ((4, 4, 10, 3), (4, 4, 4, 2), (2, 4, 2, 2)),
             ((4, 36, 2, 4), (4, 4, 4, 2), (1, 4, 2, 2)), ((2, 4, 8, 9), (16, 4, 4, 2), (8, 4, 2, 2)),
             ((4, 1, 24, 12), (24, 4, 4, 2), (12, 4, 2, 2))]


@pytest.mark.parametrize("rows,cols,deg", MANY_ROWS)
def test_many_rows_per_tile_with_two_of_four_kept(rows, cols, deg):
    """The kernel that takes all rows of a row of G_o, on batches wide enough for it (and just below): widths around its
    64-column tile, odd leading dimensions; an infinity reaches the rows that keep its row of I, and no other column."""
    w = wl.Workload("many_rows", rows, cols, deg, 333, wl.F32, 71, 72, 73, 1.0)
    enough = -(-160 // rows[0]) * 64 - 63
    for N, pad in ((enough - 1, 0), (enough, 1), (enough + 63, 0), (enough + 64, 3)):
        gh.check_parity(w, N=N, ld_pad=pad, expect_kernel=REG)
        assert (rb.rbgp_last_kernel() == "spmm_reg_rows<2>") == (N >= enough)
    N = enough + 1
    vl, Il, vf, If = gh.host_inputs(w, N)
    bad, k = Il.copy(), 21
    bad[k, 5], bad[k, N - 1], bad[k + 1, 70] = np.inf, -np.inf, np.float32(1e37)
    run = lambda X, tune=None: gh.library_spmm(w, vl, X, tune=tune, tag="many rows")[0]
    clean, got, ref = run(Il), run(bad), run(bad, (0,) * 8 + (1,))
    others = np.ones(N, bool)
    others[[5, 70, N - 1]] = False
    assert np.array_equal(got[:, others].view(np.uint32), clean[:, others].view(np.uint32))
    assert np.array_equal(got[:, [5, N - 1]] == np.inf, ref[:, [5, N - 1]] == np.inf)
    assert np.array_equal(got[:, [5, N - 1]] == -np.inf, ref[:, [5, N - 1]] == -np.inf)
    assert np.isfinite(got[:, [5, 70, N - 1]]).sum() == np.isfinite(ref[:, [5, 70, N - 1]]).sum()
    bound = 1e-6 * np.abs(ref[:, 70]).max()      # (a few rounding errors of 6e-8 of the largest sum)
    assert (np.abs(got[:, 70].astype(np.float64) - ref[:, 70]) <= bound).all()


def test_many_rows_per_tile_of_short_lists_by_batch():
    """Lists of two stages: 16 rows of G_o up to 16 column tiles and from 24 on, not where they load the XCDs unevenly, 8 rows
    from 21 tiles on."""
    for rows, widths in ((16, ((1024, True), (1025, False), (1472, False), (1473, True))), (8, ((1280, False), (1281, True)))):
        w = wl.Workload("many_rows", (rows, 4, 8, 3), (rows, 4, 4, 2), (2, 4, 2, 2), 333, wl.F32, 71, 72, 73, 1.0)
        for N, taken in widths:
            gh.check_parity(w, N=N, expect_kernel=REG)
            assert rb.rbgp_last_kernel().startswith("spmm_reg_rows<") == taken, (rows, N)


# lists of one, two and four stages; nine and three full groups of 32 rows, and four with 24 rows in the last
@pytest.mark.parametrize("rows,cols,deg", [((8, 4, 8, 9), (8, 4, 4, 2), (1, 4, 2, 2)), MANY_ROWS[1],
                                           ((4, 4, 8, 3), (8, 4, 4, 2), (4, 4, 2, 2))])
def test_many_rows_per_tile_in_tiles_of_96_columns(rows, cols, deg):
    """Batches that 64 columns a workgroup spread over 257 to 384 workgroups: the first and the last width, with odd leading
    dimensions, and one column beyond; an infinity in the last column of each block of 32 and a NaN in the last column of all."""
    w = wl.Workload("many_rows", rows, cols, deg, 333, wl.F32, 71, 72, 73, 1.0)
    tiles = 256 // rows[0]
    for N, pad in ((64 * tiles + 1, 0), (64 * tiles + 31, 1), (96 * tiles, 0), (96 * tiles + 1, 3)):
        gh.check_parity(w, N=N, ld_pad=pad, expect_kernel=REG)
        assert rb.rbgp_last_kernel() == f"spmm_reg_rows<{3 if N <= 96 * tiles else 2}>"
    N = 96 * tiles - 33
    vl, Il, _, _ = gh.host_inputs(w, N)
    bad, at = Il.copy(), [31, 63, 95, N - 1]
    bad[21, at] = [np.inf, -np.inf, np.inf, np.nan]
    run = lambda X, tune=None: gh.library_spmm(w, vl, X, tune=tune, tag="tiles of 96")[0]
    clean, got = run(Il), run(bad)
    assert rb.rbgp_last_kernel() == "spmm_reg_rows<3>"
    ref = run(bad, (0,) * 8 + (1,))
    others = np.delete(np.arange(N), at)
    assert np.array_equal(got[:, others].view(np.uint32), clean[:, others].view(np.uint32))
    for test in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(test(got[:, at]), test(ref[:, at]))


@pytest.mark.parametrize("rows,cols,deg", MANY_ROWS[:2])
def test_many_rows_per_tile_infinities_of_columns_a_row_does_not_keep(rows, cols, deg):
    """Two rows of one stage of I that are not finite in the same column: a row that keeps one of them has the sum of its own kept
    products, infinite or finite, whatever the other one holds."""
    w = wl.Workload("many_rows", rows, cols, deg, -(-160 // rows[0]) * 64, wl.F32, 71, 72, 73, 1.0)
    vl, Il, vf, _ = gh.host_inputs(w)
    bad, n = Il.copy(), 0
    at = lambda v: 64 + (4 + v) * 2 + 1          # stage 2, G_r vertex 1, G_i vertex v, G_b vertex 1
    for v in range(4):
        for u in range(4):
            if u == v:
                continue
            for x, y in ((np.inf, np.inf), (np.inf, -np.inf), (np.nan, np.inf), (np.float32(2.0 ** 110), np.inf)):
                bad[at(v), n], bad[at(u), n] = x, y
                n += 1
    got = gh.library_spmm(w, vl, bad, tag="many rows")[0][:, :n]
    assert rb.rbgp_last_kernel() == "spmm_reg_rows<2>"
    kept = rb.rbgp_mask_columns(gh.make_mask(w)).reshape(w.M, -1)
    W, X = vf.reshape(w.M, -1).astype(np.float64), bad[:, :n].astype(np.float64)
    with np.errstate(invalid="ignore"):
        ref = np.stack([W[m] @ X[kept[m]] for m in range(w.M)])
        size = np.stack([np.abs(W[m]) @ np.abs(X[kept[m]]) for m in range(w.M)])
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(got == np.inf, ref == np.inf) and np.array_equal(got == -np.inf, ref == -np.inf)
    fin = np.isfinite(ref)
    assert (np.abs(got[fin] - ref[fin]) <= 1e-6 * size[fin]).all()


# masks whose filled twin walks stages of 32 steps with at most one of k and k + 16 kept (G_i at 1/2 and 1/4, |G_b.V| of 1
# and 2), and one whose rows keep both (a complete G_i with a sparse G_b beside it)
FILLED_PAIRS = [((8, 1, 128, 1), (16, 1, 32, 1), (2, 1, 16, 1)), ((8, 1, 256, 1), (16, 1, 32, 1), (2, 1, 8, 1)),
                ((8, 2, 64, 1), (16, 1, 32, 1), (2, 1, 16, 1)), ((8, 1, 64, 2), (16, 1, 16, 2), (2, 1, 4, 2)),
                ((8, 1, 32, 4), (16, 1, 8, 4), (2, 1, 8, 2))]


@pytest.mark.parametrize("rows,cols,deg", FILLED_PAIRS)
def test_filled_masks_with_one_kept_weight_in_two_steps(rows, cols, deg):
    """The kernels of filled masks that share their columns, on the sparse MFMA where every row keeps at most one weight of
    two steps: widths around the 128-column tile; an infinity reaches the rows that keep its row of I, and of the others
    at most those of the same column."""
    w = wl.Workload("pairs", rows, cols, deg, 333, wl.F32, 61, 62, 63, 1.0)
    tune = (0,) * 8 + (3,)
    for N, pad in ((1, 0), (97, 3), (128, 0), (129, 5), (400, 4)):
        gh.check_parity(w, N=N, kernel=FILLED, tune=tune, ld_pad=pad, expect_kernel=FILLED)
        assert rb.rbgp_last_kernel() == f"spmm_reg_split_shared<{int(deg[2] < cols[2])}>"   # (the last one keeps both steps)
    N = 140
    vl, Il, vf, If = gh.host_inputs(w, N)
    bad, k = Il.copy(), 21
    bad[k, 5], bad[k, 130] = np.inf, -np.inf
    run = lambda X: gh.library_spmm(w, vl, X, kernel=FILLED, tune=tune, tag="pairs")[0]
    clean, got = run(Il), run(bad)
    others = np.ones(N, bool)
    others[[5, 130]] = False
    assert np.array_equal(got[:, others].view(np.uint32), clean[:, others].view(np.uint32))
    mask = rb.rbgp_mask_dense(gh.make_mask(w)).reshape(w.M, w.K).astype(bool)
    keeps = mask[:, k]
    W = np.zeros((w.M, w.K), np.float32)
    W[mask] = vf.reshape(-1)
    for n, sign in ((5, 1.0), (130, -1.0)):
        assert np.array_equal(got[keeps, n], np.sign(W[keeps, k]) * np.float32(sign * np.inf))
        rest = got[~keeps, n]
        assert (np.isnan(rest) | (np.abs(rest - clean[~keeps, n]) <= 1e-5 * np.abs(clean[:, n]).max())).all()


def test_filled_mask_on_a_wider_batch_allocates_nothing():
    """fp32 on a filled mask: a call on a small batch, then the capture of one wide enough for the kernels that share their
    columns, three replays on fresh inputs against the eager result."""
    import torch
    rows, cols, deg = FILLED_PAIRS[0]
    w = wl.Workload("pairs_graph", rows, cols, deg, 2560, wl.F32, 61, 62, 63, 1.0)
    mask = gh.make_mask(w)
    rb.rbgp_mask_set_kernel(mask, FILLED)
    stream = lambda: torch.cuda.current_stream().cuda_stream
    packed = torch.zeros(rb.rbgp_packed_bytes(mask, w.dtype), dtype=torch.uint8, device="cuda:0")
    rb.rbgp_pack(mask, w.dtype, wl.kept_weights(w), packed.data_ptr(), stream())
    I = torch.zeros((w.K, w.N), device="cuda:0")
    O = torch.zeros((w.M, w.N), device="cuda:0")
    call = lambda n: rb.rbgp_spmm(mask, w.dtype, w.M, w.K, n, packed.data_ptr(), I.data_ptr(), w.N, O.data_ptr(), w.N, stream())
    call(40)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(w.N)
    for seed in (1, 2, 3):
        I.copy_(torch.randn(I.shape, device="cuda:0", generator=torch.Generator(device="cuda:0").manual_seed(seed)))
        call(w.N)
        assert rb.rbgp_last_kernel() == "spmm_reg_split_shared<1>"
        torch.cuda.synchronize()
        want = O.clone()
        O.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(O, want)


@pytest.mark.parametrize("rows,cols,deg", [((4, 4, 32, 1), (8, 1, 32, 1), (4, 1, 8, 1)), ((4, 1, 32, 4), (8, 3, 32, 1), (2, 3, 16, 1)),
                                           ((2, 2, 64, 2), (4, 2, 16, 2), (2, 2, 4, 2)), ((4, 4, 8, 4), (8, 1, 8, 4), (4, 1, 8, 2))])
def test_lds_family_split_operands(rows, cols, deg):
    """RBGP_TUNE_SPLIT_OPERANDS on the LDS family: widths around the tile of two groups of waves, one and two groups of G_i
    vertices, 8 and 16 kept steps; infinities and tiny operands as the fp32 kernel gives them."""
    w = wl.Workload("lds_split", rows, cols, deg, 333, wl.F32, 11, 12, 13, 1.0)
    forced, never = (0,) * 8 + (2,), (0,) * 8 + (1,)
    for N, pad in ((4, 0), (100, 4), (128, 0), (129, 3), (300, 0)):
        gh.check_parity(w, N=N, kernel=MFMA, tune=forced, ld_pad=pad, expect_kernel=MFMA)
        assert rb.rbgp_last_kernel() == f"spmm_mfma_split<{deg[2] * deg[3]}, {int(deg[2] < cols[2])}, 2, 2>"
    N = 132
    vl, Il, vf, If = gh.host_inputs(w, N)
    bad = Il.copy()
    bad[3, 5], bad[7, 60], bad[40, 130], bad[41, 131] = np.inf, np.nan, -np.inf, np.float32(3.4e38)
    bad[:, 100] *= np.float32(2.0 ** -120)
    run = lambda X, tune: gh.library_spmm(w, vl, X, kernel=MFMA, tune=tune, tag="split operands")[0]
    clean, got, ref = run(Il, forced), run(bad, forced), run(bad, never)
    others = np.ones(N, bool)
    others[[5, 60, 100, 130, 131]] = False
    assert np.array_equal(got[:, others].view(np.uint32), clean[:, others].view(np.uint32))
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
    fin = np.isfinite(ref)
    scale = np.abs(np.where(fin, ref, 0)).max(axis=0)       # (column by column: a few rounding errors of 6e-8 of its sums)
    assert (np.abs(np.where(fin, got, 0).astype(np.float64) - np.where(fin, ref, 0)) <= 1e-6 * scale).all()


# 8 and 16 kept steps on the sparse form, 8 and 16 on the dense one (vertices that keep both k and k + 16); four workgroups a column tile
SPLIT_FORMS = [((4, 4, 32, 1), (8, 1, 32, 1), (4, 1, 8, 1), "8, 1"), ((2, 1, 64, 4), (4, 3, 32, 1), (2, 3, 16, 1), "16, 1"),
               ((4, 4, 2, 16, 1), (8, 1, 2, 16, 1), (4, 1, 2, 4, 1), "8, 0"), ((4, 4, 8, 4), (8, 1, 8, 4), (4, 1, 8, 2), "16, 0")]


@pytest.mark.parametrize("form,N", [("2, 2", 132), ("2, 1", 4196), ("4, 1", 13092)])
@pytest.mark.parametrize("rows,cols,deg,steps", SPLIT_FORMS)
def test_lds_family_split_operands_in_every_form(rows, cols, deg, steps, form, N):
    """Two groups of waves on 64 columns a workgroup, one, and one on 128: the sums of the fp32 kernel, and its bits in columns with
    infinities, operands of 2^105 and more or nothing that is a number, one in every column block of a tile and in the last."""
    w = wl.Workload("split_forms", rows, cols, deg, N, wl.F32, 41, 42, 43, 1.0, **({"roles": (0, 1, 2, 2, 3)} if len(rows) == 5 else {}))
    run = lambda X, v: gh.library_spmm(w, vl, X, kernel=MFMA, tune=(0,) * 8 + (v,), tag="every form")[0]
    vl, Il, vf, If = gh.host_inputs(w, N)
    bad, cols_bad = Il.copy(), [5, 37, 70, 101, 128, N - 40, N - 1]
    bad[3, 5], bad[w.K - 1, 70], bad[:, 101], bad[17, N - 1] = np.inf, -np.inf, np.nan, np.float32(3e38)
    bad[:, [37, 128, N - 40]] *= np.float32(2.0 ** 110)
    clean, got = run(Il, 2), run(bad, 2)
    assert rb.rbgp_last_kernel() == f"spmm_mfma_split<{steps}, {form}>"
    plain, ref = run(Il, 1), run(bad, 1)
    assert rb.rbgp_last_kernel() == "spmm_mfma"
    assert (np.abs(clean.astype(np.float64) - plain) <= 1e-6 * np.abs(plain).max(axis=0)).all()   # (a few rounding errors of 6e-8)
    others = np.delete(np.arange(N), cols_bad)
    assert np.array_equal(got[:, others].view(np.uint32), clean[:, others].view(np.uint32))
    assert np.isfinite(ref[:, 37]).all()
    for n in cols_bad:   # (tiles without the operand of 3e38 keep the split's sums)
        same = got[:, n].view(np.uint32) == ref[:, n].view(np.uint32)
        kept = got[:, n].view(np.uint32) == clean[:, n].view(np.uint32)
        assert (same | kept | np.isnan(got[:, n]) & np.isnan(ref[:, n])).all()
        assert same.all() or n not in (37, 128, N - 40)


@pytest.mark.parametrize("rows,cols,deg", [((4, 4, 32, 1), (8, 1, 32, 1), (4, 1, 8, 1)), ((4, 1, 64, 4), (8, 3, 32, 1), (2, 3, 16, 1)),
                                           ((2, 2, 64, 2), (4, 2, 16, 2), (2, 2, 4, 2))])
def test_lds_family_split_operands_repair_sums_as_the_fp32_kernel(rows, cols, deg):
    """Columns that split operands cannot give (infinities, operands of 2^105 and more with finite sums, columns that are
    not numbers throughout, the last column of a partly empty tile): the sums are the fp32 kernel's, bit for bit."""
    w = wl.Workload("lds_repair", rows, cols, deg, 333, wl.F32, 41, 42, 43, 1.0)
    run = lambda X, v: gh.library_spmm(w, vl, X, kernel=MFMA, tune=(0,) * 8 + (v,), tag="repaired sums")[0]
    for N in (64, 132, 300):
        vl, Il, vf, If = gh.host_inputs(w, N)
        bad, cols_bad = Il.copy(), [0, 5, 31, 37, 63, N - 1]
        bad[3, 0], bad[w.K - 1, 5], bad[:, 31] = np.inf, -np.inf, np.nan
        bad[:, [37, 63]] *= np.float32(2.0 ** 110)
        bad[17, N - 1] = np.float32(3e38)
        clean, got, ref = run(Il, 2), run(bad, 2), run(bad, 1)
        others = np.ones(N, bool)
        others[cols_bad] = False
        assert np.array_equal(got[:, others].view(np.uint32), clean[:, others].view(np.uint32))
        assert np.isfinite(ref[:, 37]).all()
        for n in cols_bad:   # (tiles without the operand of 3e38 keep the split's sums)
            same = got[:, n].view(np.uint32) == ref[:, n].view(np.uint32)
            kept = got[:, n].view(np.uint32) == clean[:, n].view(np.uint32)
            assert (same | kept | np.isnan(got[:, n]) & np.isnan(ref[:, n])).all()
            assert same.all() or n not in (37, 63)


def test_lds_family_split_operands_repair_costs_a_few_products():
    """A product whose inputs are not numbers at all, or in one column, takes a few times an ordinary one's time: the
    repair runs on the matrix core, a stage's loads ahead (a serial loop took 15 and 5 times)."""
    import torch
    w = wl.sdmm4096_table2(2, 2)
    N = 1536
    mask = rb.rbgp_make_mask(w.rows, w.cols, w.row_deg, w.mask_seed)
    rb.rbgp_mask_set_kernel(mask, MFMA)
    stream = torch.cuda.current_stream().cuda_stream
    packed = torch.randn(rb.rbgp_packed_bytes(mask, rb.F32) // 4, device="cuda:0")
    I, O = torch.rand((w.K, N), device="cuda:0"), torch.empty((w.M, N), device="cuda:0")

    def microseconds():
        times = []
        for _ in range(9):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            for _ in range(10):
                rb.rbgp_spmm(mask, rb.F32, w.M, w.K, N, packed.data_ptr(), I.data_ptr(), N, O.data_ptr(), N, stream)
            e[1].record()
            torch.cuda.synchronize()
            times.append(100 * e[0].elapsed_time(e[1]))
        return sorted(times)[4]

    usual = microseconds()
    I[5, 77] = float("inf")
    one = microseconds()
    I.fill_(float("nan"))
    every = microseconds()
    print(f"[gpu] us: {usual:.0f}, one infinity {one:.0f}, not a number throughout {every:.0f}", flush=True)
    assert torch.isnan(O).all()
    assert one < 3.5 * usual and every < 7 * usual


@pytest.mark.parametrize("dtype,variant", [(wl.F32, 2), (wl.F32, 3), (wl.BF16, 2), (wl.BF16, 4)])
def test_padding_steps_of_row_pairs_read_nothing(dtype, variant):
    """Rows of I so far apart that the rows of one stage and the columns of the next one pass 2^31 bytes: the padding
    steps of a stage (20 of 32 are real) must not bring an infinity of another row and column into the sums."""
    import torch
    w = wl.Workload("wide_rows", (2, 128, 2, 1), (2, 1, 10, 2), (1, 1, 10, 2), 400, dtype, 31, 32, 33, 1.0)
    N, es = 400, 2 if dtype == wl.BF16 else 4
    ld = (2 ** 31 // es - 200) // 20 // 8 * 8              # (a stage spans 20 rows)
    assert (20 * ld + 128) * es < 2 ** 31 < (20 * ld + N) * es
    vl, Il, vf, If = gh.host_inputs(w, N)
    mask = gh.make_mask(w)
    rb.rbgp_mask_set_kernel(mask, REG)
    rb.rbgp_mask_tune(mask, rb.TUNE_SPLIT_OPERANDS if dtype == wl.F32 else rb.TUNE_SHARED_COLUMNS, variant)
    stream = torch.cuda.current_stream().cuda_stream
    packed = torch.zeros(rb.rbgp_packed_bytes(mask, dtype), dtype=torch.uint8, device="cuda:0")
    rb.rbgp_pack(mask, dtype, np.ascontiguousarray(vl), packed.data_ptr(), stream)
    I = torch.zeros((w.K, ld), dtype=torch.float32 if dtype == wl.F32 else torch.int16, device="cuda:0")
    I[:, :N] = torch.from_numpy(Il.view(np.int16) if dtype == wl.BF16 else Il).to("cuda:0")
    col = 2 ** 31 // es - 20 * ld + 40                      # what a step at byte 2^31 would read for column 40
    I[20, col] = float("inf") if dtype == wl.F32 else 0x7F80
    O = torch.full((w.M, N), float("nan"), dtype=torch.float32, device="cuda:0")
    print(f"[gpu] padding steps, rows of {ld} elements, variant {variant}", flush=True)
    rb.rbgp_spmm(mask, dtype, w.M, w.K, N, packed.data_ptr(), I.data_ptr(), ld, O.data_ptr(), N, stream)
    out = O.cpu().numpy()
    ref, den = gh.oracle_spmm(w, vf, If)
    others = np.arange(N) != col
    assert col < N
    assert np.isfinite(out[:, others]).all()
    assert orc.normalised_error(out[:, others], ref[:, others], den[:, others]) <= 4e-6


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
def test_kernels_of_row_pairs_on_the_fused_convolution(dtype):
    """The 3x3 convolution through the split-operand and the shared-column kernels: images of 8 and 16 columns, a last
    column tile that is partly empty."""
    w = wl.Workload("pairs_conv", (4, 128, 1, 1), (4, 2, 1, 9), (2, 2, 1, 9), 333, dtype, 7, 8, 9, 1.0)
    tunes = [(0,) * 8 + (v,) for v in (2, 3)] if dtype == wl.F32 else [(0,) * 9 + (v,) for v in (2, 3, 4, 5, 6)]
    for B, H, W in ((3, 5, 8), (2, 16, 16)):
        vals, X = wl.kept_weights(w), wl.conv_activations(w, B, H, W)
        vl, Xl, vf, Xf = gh.host_inputs(w, vals=vals, I=X)
        ref, den = gh.oracle_spmm(w, vf, orc.im2col_3x3(Xf))
        for tune in tunes:
            out = gh.library_conv3x3(w, vl, Xl, tune=tune)
            assert orc.normalised_error(out, ref, den) <= 4e-6


# more than 16 rows per column set with a composite |G_b.U|: the register family runs on the same mask factored as
# G_o (x) G_r (x) (G_i (x) J(q, 1)) (x) J(|G_b.U| / q, .), whose MFMA groups are fuller.  (rows, cols, degrees, rows per
# group before and after)
REGROUP_SHAPES = [
    ((4, 4, 2, 9), (4, 4, 4, 2), (2, 4, 2, 2), 9, 12),      # a transposed 3x3 layer: 36 rows, 4 x 9 -> 3 x 12
    ((4, 8, 2, 9), (4, 2, 2, 2), (2, 2, 1, 2), 9, 12),      # 72 rows: 8 x 9 -> 6 x 12, stages of 4 steps in 8
    ((2, 32, 1, 9), (2, 4, 2, 2), (1, 4, 2, 2), 9, 16),     # 288 rows: 32 x 9 -> 18 x 16
    ((4, 4, 4, 12), (4, 2, 4, 3), (2, 2, 2, 3), 12, 16),    # 48 rows: 4 x 12 -> 3 x 16
]


@pytest.mark.parametrize("idx", range(len(REGROUP_SHAPES)))
@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
def test_register_family_on_the_regrouped_mask(idx, dtype):
    rows, cols, deg, before, after = REGROUP_SHAPES[idx]
    N = 333 if dtype == wl.F32 else 328
    w = wl.Workload(f"regroup{idx}", rows, cols, deg, N, dtype, 250 + idx, 260 + idx, 270 + idx, 1.0)
    mask = rb.rbgp_make_mask(rows, cols, deg, w.mask_seed)
    plan = rb.rbgp_mask_reg_plan(mask)
    assert plan[14] == after                      # rows of the MFMA group in use on the regrouped mask
    rb.rbgp_mask_check_tables(mask)
    gh.check_parity(w, kernel=REG, ld_pad=3 if dtype == wl.F32 else 8, expect_kernel=REG)
    gh.check_parity(w, N=64, kernel=REG, expect_kernel=REG)
    gh.check_parity(w, N=2312, kernel=REG, tune=(0, 0, 0, 0, 0, 1), expect_kernel=REG)
    gh.check_parity(w, N=200, kernel=REG, tune=(0, 0, 0, 0, 0, 2), expect_kernel=REG)
    gh.check_parity(w, kernel=rb.KERNEL_AUTO)
    gh.check_parity(w, kernel=GEN, expect_kernel=GEN)   # the generic family runs the mask as given: same results


# a complete G_o: the register family runs on the same mask with G_o (x) G_r merged into one tile column, whose
# stages are longer (rows, cols, degrees, steps per stage before and after)
MERGED_COLUMN_SHAPES = [
    ((4, 2, 2, 4), (4, 2, 4, 2), (4, 2, 2, 2), 8, 32),          # 4 tiles of 8 steps -> one stage of 32
    ((8, 2, 2, 2), (8, 1, 4, 4), (8, 1, 2, 4), 8, 72),          # 8 tiles of 8 steps -> one stage of 64 in 72
    ((8, 1, 4, 1), (8, 2, 4, 2), (8, 2, 2, 2), 8, 72),          # one row per column set
    ((2, 4, 1, 2), (128, 1, 1, 2), (128, 1, 1, 2), 8, 72),      # 128 tiles of 2 steps in 8 -> 4 stages of 64 in 72
    ((4, 4, 8, 1), (32, 1, 8, 1), (32, 1, 2, 1), 8, 72),        # Table 2's shape with a complete G_o, small
]


@pytest.mark.parametrize("idx", range(len(MERGED_COLUMN_SHAPES)))
@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
def test_register_family_on_the_mask_with_merged_tile_columns(idx, dtype):
    rows, cols, deg, before, after = MERGED_COLUMN_SHAPES[idx]
    N = 333 if dtype == wl.F32 else 328
    w = wl.Workload(f"merged{idx}", rows, cols, deg, N, dtype, 280 + idx, 290 + idx, 295 + idx, 1.0)
    mask = rb.rbgp_make_mask(rows, cols, deg, w.mask_seed)
    plan = rb.rbgp_mask_reg_plan(mask)
    assert plan[2] == before and plan[14] > 0 and plan[15] > 0
    rb.rbgp_mask_check_tables(mask)
    gh.check_parity(w, kernel=REG, ld_pad=3 if dtype == wl.F32 else 8, expect_kernel=REG)
    gh.check_parity(w, N=64 if dtype == wl.F32 else 128, kernel=REG, expect_kernel=REG)
    gh.check_parity(w, N=2312, kernel=REG, tune=(0, 0, 0, 0, 0, 1), expect_kernel=REG)
    gh.check_parity(w, N=200, kernel=REG, tune=(0, 0, 0, 0, 0, 2), expect_kernel=REG)
    gh.check_parity(w, kernel=GEN, expect_kernel=GEN)


def test_regrouped_masks_randomised():
    """Seeded random masks with a composite |G_b.U| and up to 16 x 15 rows per column set, fp32, register family:
    the result is the oracle's whether or not the library regroups the mask; at least a third of them are regrouped."""
    g = np.random.Generator(np.random.PCG64(20))
    ran = regrouped = 0
    for it in range(60):
        a_o, c_o = int(g.choice([2, 4, 8])), int(g.choice([2, 4, 8]))
        d_o = int(g.choice([x for x in (1, 2, 4, 8) if x <= c_o]))
        a_r, c_r = int(g.choice([2, 4, 8, 16])), int(g.choice([1, 2, 4]))
        a_i, c_i = int(g.choice([1, 2, 4])), int(g.choice([1, 2, 4]))
        d_i = int(g.choice([x for x in (1, 2, 4) if x <= c_i]))
        a_b, c_b = int(g.choice([4, 6, 8, 9, 10, 12, 15])), int(g.choice([1, 2, 3]))
        rows, cols, deg = (a_o, a_r, a_i, a_b), (c_o, c_r, c_i, c_b), (d_o, c_r, d_i, c_b)
        try:
            mask = rb.rbgp_make_mask(rows, cols, deg, 300 + it)
        except rb.RbgpError:
            continue                                  # (not a shape the sampler accepts)
        plan = rb.rbgp_mask_reg_plan(mask)
        if plan[0] == 0:
            continue
        rb.rbgp_mask_check_tables(mask)
        w = wl.Workload(f"regroup_rand{it}", rows, cols, deg, int(g.choice([64, 200, 333])), wl.F32, 300 + it, 301 + it,
                        302 + it, 1.0)
        gh.check_parity(w, kernel=REG, ld_pad=int(g.choice([0, 3])), expect_kernel=REG)
        ran += 1
        regrouped += plan[14] > 0
    assert ran >= 30 and 3 * regrouped >= ran


def test_fp32_row_groups_on_the_fused_convolution_and_refusals():
    # a density-1/2 VGG19 layer shape (complete G_i joins G_r: 32 rows per column set), images 8 pixels wide: tap-grouped
    w = wl.Workload("rowgroups_conv", (4, 4, 4, 2), (4, 2, 8, 9), (2, 2, 8, 9), 0, wl.F32, 71, 72, 73, 1.0)
    X = wl.conv_activations(w, 6, 8, 8)
    want, den = gh.oracle_spmm(w, wl.kept_weights(w), orc.im2col_3x3(X))
    for ng in (1, 2):
        for sets in (1, 2):
            out = gh.library_conv3x3(w, wl.kept_weights(w), X, tune=(0, 0, 0, 0, ng, 0, 0, sets), kernel=REG)
            assert orc.normalised_error(out, want, den) <= gh.TOL[w.dtype]
    # a mask with 8 rows per column set has no such groups
    with pytest.raises(rb.RbgpError) as e:
        gh.check_parity(wl.VGG19_CONV5, N=256, kernel=REG, tune=(0, 0, 0, 0, 2), expect_kernel=REG)
    assert e.value.code == rb.EUNSUPPORTED


# stages of 8 contraction steps, every stage list of the same length (a multiple of 4): waves that take several
# column tiles one after the other.  (rows, cols, degrees, column tiles per wave to try, row groups per wave)
COLUMN_TILE_SHAPES = [
    ((8, 4, 4, 9), (8, 4, 2, 2), (4, 4, 1, 2), (2, 4, 8), 1),    # a transposed 3x3 layer: 36 rows -> 4 x 9, lists of 4
    ((8, 4, 4, 11), (8, 4, 2, 2), (4, 4, 1, 2), (2, 4), 2),      # 44 rows -> 4 x 11: two of the four tile rows per wave
    ((8, 4, 4, 9), (8, 3, 4, 2), (4, 3, 1, 2), (4,), 1),         # stages of 6 steps in 8
]


@pytest.mark.parametrize("idx", range(len(COLUMN_TILE_SHAPES)))
def test_fp32_register_family_column_tiles_per_wave(idx):
    """RBGP_TUNE_COLUMN_TILES: N of one tile, of several waves' worth with a ragged last tile and a last wave that has
    fewer tiles than the others, padded leading dimension."""
    rows, cols, deg, tiles, ng = COLUMN_TILE_SHAPES[idx]
    w = wl.Workload(f"coltiles{idx}", rows, cols, deg, 333, wl.F32, 140 + idx, 150 + idx, 160 + idx, 1.0)
    for ct in tiles:
        tune = (0, 0, 0, 0, ng, 1, ct)   # (no split of the stage lists, which small N would bring)
        gh.check_parity(w, kernel=REG, tune=tune, ld_pad=3, expect_kernel=REG)          # 6 tiles
        gh.check_parity(w, N=64, kernel=REG, tune=tune, expect_kernel=REG)              # one tile
        gh.check_parity(w, N=2309, kernel=REG, tune=tune, ld_pad=1, expect_kernel=REG)  # 37 tiles


def test_column_tiles_per_wave_refusals_and_default():
    # stage lists of different lengths (sparse G_o, two tile rows per group: no kernel of this kind), a split list,
    # stages of more than 8 steps, bf16: refused
    ragged = wl.Workload("coltiles_ragged", (16, 2, 2, 4), (16, 2, 4, 2), (8, 2, 2, 2), 256, wl.F32, 171, 172, 173, 1.0)
    long_steps = wl.Workload("coltiles_18", (8, 4, 4, 9), (8, 4, 4, 2), (4, 4, 2, 2), 256, wl.F32, 174, 175, 176, 1.0)
    ok = wl.Workload("coltiles_ok", (8, 4, 4, 9), (8, 4, 2, 2), (4, 4, 1, 2), 256, wl.F32, 177, 178, 179, 1.0)
    for w, tune in ((ragged, (0, 0, 0, 0, 0, 1, 2)), (long_steps, (0, 0, 0, 0, 0, 1, 2)), (ok, (0, 0, 0, 0, 0, 2, 2)),
                    (ok, (0, 0, 0, 0, 0, 1, 3)), (ok, (0, 0, 0, 0, 0, 1, 32)), (replace(ok, dtype=wl.BF16), (0, 0, 0, 0, 0, 1, 2))):
        with pytest.raises(rb.RbgpError) as e:
            gh.check_parity(w, kernel=REG, tune=tune, expect_kernel=REG)
        assert e.value.code == rb.EUNSUPPORTED
    # the library's own choice on the backward data product of the headline layer (64 tile rows of 9 rows, 8 stages of
    # 8 steps): whatever it takes, the result is the oracle's
    gh.check_parity(ok, N=8192, kernel=rb.KERNEL_AUTO)


# stages of 72 steps with 2, 4, 8 and 16 weight rows per tile row: the kernels with one register set (two waves per SIMD)
ONE_SET_SHAPES = [((4, 1, 4, 2), 2), ((4, 2, 4, 2), 4), ((4, 4, 4, 2), 8), ((4, 4, 4, 4), 16)]


# stages of 72, 36, 32 and 18 steps: columns and left degrees of the factors
ONE_SET_STAGES = {72: ((4, 4, 4, 9), (2, 4, 2, 9)), 36: ((4, 2, 4, 9), (2, 2, 2, 9)), 32: ((4, 4, 4, 4), (2, 4, 2, 4)),
                  18: ((4, 1, 4, 9), (2, 1, 2, 9))}


@pytest.mark.parametrize("idx", range(len(ONE_SET_SHAPES)))
@pytest.mark.parametrize("steps", sorted(ONE_SET_STAGES))
def test_fp32_register_family_one_register_set(idx, steps):
    """RBGP_TUNE_REGISTER_SETS = 1: ragged N, padded leading dimension, one column tile, a split stage list."""
    rows, rs = ONE_SET_SHAPES[idx]
    cols, deg = ONE_SET_STAGES[steps]
    w = wl.Workload(f"oneset{steps}_{idx}", rows, cols, deg, 333, wl.F32, 180 + idx, 190 + idx, 200 + idx, 1.0)
    plan = rb.rbgp_mask_reg_plan(rb.rbgp_make_mask(w.rows, w.cols, w.row_deg, w.mask_seed))
    assert 16 // plan[0] == rs and plan[2] == steps
    pairing = 1 if rs == 8 else 0   # (8 rows: the fixed pairs, not the tile-by-tile pairing kernel)
    for N, split, pad in ((333, 1, 3), (64, 0, 0), (2309, 1, 1), (200, 2, 0), (130, 4, 2)):
        gh.check_parity(w, N=N, kernel=REG, tune=(0, 0, 0, pairing, 0, split, 0, 1), ld_pad=pad, expect_kernel=REG)
    gh.check_parity(w, N=333, kernel=REG, tune=(0, 0, 0, pairing, 0, 0, 0, 2), expect_kernel=REG)


@pytest.mark.parametrize("idx", range(len(ONE_SET_SHAPES)))
@pytest.mark.parametrize("steps", [72, 36])
def test_bf16_register_family_one_register_set(idx, steps):
    """The bf16 kernels with one register set (128-column tiles, one or two row groups, stages of 72 and 36 steps):
    ragged N, a split stage list, the bf16-output mode; 64-column tiles have no such variant."""
    rows, rs = ONE_SET_SHAPES[idx]
    cols, deg = ((4, 4, 4, 9), (2, 4, 2, 9)) if steps == 72 else ((4, 2, 4, 9), (2, 2, 2, 9))
    w = wl.Workload(f"oneset_bf16_{steps}_{idx}", rows, cols, deg, 328, wl.BF16, 210 + idx, 220 + idx, 230 + idx, 1.0)
    assert rb.rbgp_mask_reg_plan(rb.rbgp_make_mask(w.rows, w.cols, w.row_deg, w.mask_seed))[2] == steps
    for N, groups, split in ((328, 1, 1), (1096, 2, 1), (136, 1, 2), (2312, 2, 4), (128, 1, 0)):
        gh.check_parity(w, N=N, kernel=REG, tune=(0, 128, 0, 0, groups, split, 0, 1), expect_kernel=REG)
    # bf16 output: the rounding of what the fp32-output mode of the same launch stores
    vl, Il, vf, If = gh.host_inputs(w, 328)
    out16, _ = gh.library_spmm(w, vl, Il, REG, (0, 128, 0, 0, 1, 1, 0, 1), out_bf16=True)
    out32, _ = gh.library_spmm(w, vl, Il, REG, (0, 128, 0, 0, 1, 1, 0, 1))
    assert np.array_equal((out16.view(np.uint32) >> 16).astype(np.uint16), orc.f32_to_bf16_bits(out32))
    with pytest.raises(rb.RbgpError) as e:
        gh.check_parity(w, N=328, kernel=REG, tune=(0, 64, 0, 0, 1, 1, 0, 1), expect_kernel=REG)
    assert e.value.code == rb.EUNSUPPORTED
    if rs == 16:   # four groups per wave: built for stages of up to 36 steps
        if steps == 36:
            gh.check_parity(w, N=1096, kernel=REG, tune=(0, 128, 0, 0, 4, 1, 0, 1), expect_kernel=REG)
        else:
            with pytest.raises(rb.RbgpError) as e:
                gh.check_parity(w, N=1096, kernel=REG, tune=(0, 128, 0, 0, 4, 1, 0, 1), expect_kernel=REG)
            assert e.value.code == rb.EUNSUPPORTED


def test_bf16_one_register_set_on_short_stages():
    """Stages of 32 and 18 steps: with two groups only where a wave has a single stage, with four groups always."""
    one_stage32 = wl.Workload("oneset_bf16_single32", (4, 4, 2, 2), (1, 4, 4, 2), (1, 4, 4, 2), 1096, wl.BF16, 241, 242, 243, 1.0)
    one_stage18 = wl.Workload("oneset_bf16_single18", (4, 2, 4, 2), (1, 2, 4, 4), (1, 2, 2, 4), 1096, wl.BF16, 244, 245, 246, 1.0)
    for w in (one_stage32, one_stage18):
        for sets in (1, 2, 0):
            gh.check_parity(w, kernel=REG, tune=(0, 128, 0, 0, 2, 1, 0, sets), expect_kernel=REG)
    gh.check_parity(one_stage32, kernel=REG, tune=(0, 128, 0, 0, 4, 1, 0, 1), expect_kernel=REG)
    several = wl.Workload("oneset_bf16_several18", (4, 4, 4, 4), (4, 1, 4, 9), (2, 1, 2, 9), 1096, wl.BF16, 247, 248, 249, 1.0)
    gh.check_parity(several, kernel=REG, tune=(0, 128, 0, 0, 4, 1, 0, 1), expect_kernel=REG)
    with pytest.raises(rb.RbgpError) as e:
        gh.check_parity(several, kernel=REG, tune=(0, 128, 0, 0, 2, 1, 0, 1), expect_kernel=REG)
    assert e.value.code == rb.EUNSUPPORTED


def test_one_register_set_on_the_headline_layer_and_refusals():
    gh.check_parity(wl.VGG19_CONV5, N=512, kernel=REG, tune=(0, 0, 0, 1, 0, 0, 0, 1), expect_kernel=REG)
    # the fused convolution on 4-pixel-wide images (no tap grouping): the same kernel reading the activations
    w = wl.VGG19_CONV5
    X = wl.conv_activations(w, 9, 4, 4)
    want, den = gh.oracle_spmm(w, wl.kept_weights(w), orc.im2col_3x3(X))
    for sets in (1, 2):
        out = gh.library_conv3x3(w, wl.kept_weights(w), X, tune=(0, 0, 0, 1, 0, 0, 0, sets), kernel=REG)
        assert orc.normalised_error(out, want, den) <= gh.TOL[w.dtype]
    short = wl.Workload("oneset_8", (8, 4, 4, 9), (8, 4, 2, 2), (4, 4, 1, 2), 256, wl.F32, 174, 175, 176, 1.0)
    for w, tune in ((short, (0, 0, 0, 0, 0, 0, 0, 1)),                       # stages of 8 steps
                    (wl.VGG19_CONV5, (0, 0, 0, 2, 0, 0, 0, 1)),              # with the tile-by-tile pairing kernel
                    (wl.VGG19_CONV5, (0, 0, 0, 1, 0, 0, 0, 3)),              # not a value of the knob
                    (replace(wl.VGG19_CONV3_BF16, N=256), (0, 64, 0, 0, 0, 0, 0, 1))):   # bf16 on 64-column tiles
        with pytest.raises(rb.RbgpError) as e:
            gh.check_parity(w, N=256, kernel=REG, tune=tune, expect_kernel=REG)
        assert e.value.code == rb.EUNSUPPORTED


@pytest.mark.parametrize("sets", [1, 2])
@pytest.mark.parametrize("N", [1021, 1025, 1537, 1984])
def test_register_sets_where_the_default_pairs_tile_rows(N, sets):
    """RBGP_TUNE_REGISTER_SETS by itself below 1024 stage lists (conv5: 32 a tile of 64 columns) runs the kernel that has the knob,
    also at sizes where the default pairs tile rows (from 513 lists on); with one set refused, as ever, where every list is paired."""
    tune = (0,) * 7 + (sets,)
    gh.check_parity(wl.VGG19_CONV5, N=N, kernel=REG, expect_kernel=REG)
    assert rb.rbgp_last_kernel() == ("spmm_reg_dual" if N > 1024 else "spmm_reg")
    gh.check_parity(wl.VGG19_CONV5, N=N, kernel=REG, tune=tune, expect_kernel=REG)
    assert rb.rbgp_last_kernel() == "spmm_reg"
    if sets == 1 and N == 1984:
        with pytest.raises(rb.RbgpError) as e:
            gh.check_parity(wl.VGG19_CONV5, N=1985, kernel=REG, tune=tune)
        assert e.value.code == rb.EUNSUPPORTED


def test_activations_beyond_4_gib():
    """An I of 4.6 GB (WRN shape, 2 000 037 columns, odd leading dimension): the kernels'
    32-bit offsets must only span one stage.  A sample of output columns is checked."""
    w = replace(wl.WRN_G1, N=2_000_037, name="wrn_4gib")
    vl, Il, vf, If = gh.host_inputs(w)
    cols = np.r_[0:64, 1_000_000:1_000_064, 1_999_936:2_000_037]
    ref, den = gh.oracle_spmm(w, vf, np.ascontiguousarray(If[:, cols]))
    for kernel in (rb.KERNEL_AUTO, MFMA, GEN):
        out, used = gh.library_spmm(w, vl, Il, kernel=kernel, tune=(1, 64, 0) if kernel == MFMA else None,
                                    ld_pad=3 if kernel == MFMA else 0, tag="beyond 4 GiB")
        assert used == (REG if kernel == rb.KERNEL_AUTO else kernel)
        err = orc.normalised_error(out[:, cols], ref, den)
        assert err <= gh.TOL[w.dtype], err
        assert np.all(np.isfinite(out[:, ::4099]))


# ------------------------------------------------------------------ fused 3x3 convolution
CONV_CASES = [
    # workload (K = 9 * channels), images, height, width
    (wl.Workload("conv_small", (4, 2, 2, 4), (4, 2, 4, 9), (2, 2, 4, 9), 0, wl.F32, 61, 62, 63, 1.0), 3, 4, 8),
    (wl.Workload("conv_ragged", (4, 1, 4, 3), (4, 2, 4, 9), (2, 2, 2, 9), 0, wl.F32, 64, 65, 66, 1.0), 5, 3, 4),
    (wl.Workload("conv_wide", (4, 2, 4, 1), (4, 2, 4, 9), (2, 2, 2, 9), 0, wl.F32, 67, 68, 69, 1.0), 2, 5, 32),
    (wl.VGG19_CONV5, 128, 4, 4),          # the headline layer: 512 -> 512 channels, 4x4 pixels, batch 128
    (wl.WRN_G1, 8, 32, 32),               # WRN-40-4 group 1 at batch 8
    (wl.VGG19_CONV3_BF16, 128, 8, 8),     # bf16: 256 -> 256 channels, 8x8 pixels (128-column wave tiles)
    (replace(wl.VGG19_CONV3_BF16, name="conv3_bf16_4x4"), 33, 4, 4),     # bf16, 64-column tiles, ragged N
    (replace(wl.Workload("conv_small_bf16", (4, 2, 2, 4), (4, 2, 4, 9), (2, 2, 4, 9), 0, wl.BF16, 71, 72, 73, 1.0)), 3, 5, 8),
    # stages padded to the next kernel size: 54 -> 72 steps, 9 -> 18 steps, 27 -> 36 steps with 16 rows per tile row
    (wl.Workload("conv_pad54", (4, 2, 4, 1), (4, 1, 12, 9), (2, 1, 6, 9), 0, wl.F32, 74, 75, 76, 1.0), 2, 4, 8),
    (wl.Workload("conv_pad9_bf16", (4, 1, 2, 1), (4, 1, 2, 9), (2, 1, 1, 9), 0, wl.BF16, 77, 78, 79, 1.0), 3, 3, 12),
    (wl.Workload("conv_pad27_r16", (4, 4, 4, 4), (4, 3, 4, 9), (2, 3, 1, 9), 0, wl.F32, 80, 81, 82, 1.0), 2, 4, 16),
]


@pytest.mark.parametrize("case", CONV_CASES, ids=lambda c: c[0].name)
def test_fused_conv3x3_equals_spmm_on_the_lowered_input(case):
    """rbgp_conv3x3 on padded activations = the oracle's product with the explicitly
    lowered input (im2col written out in the oracle)."""
    w, B, H, W = case
    vals = wl.kept_weights(w)
    X = wl.conv_activations(w, B, H, W)
    if w.dtype == wl.BF16:                # both sides consume the same bf16 bits
        vals_lib, X_lib = wl.to_bf16_bits(vals), wl.to_bf16_bits(X)
        vals, X = wl.bf16_bits_as_f32(vals_lib), wl.bf16_bits_as_f32(X_lib)
    else:
        vals_lib, X_lib = vals, X
    ref, den = gh.oracle_spmm(w, vals, orc.im2col_3x3(X))
    tunes = [None, (0, 0, 0, 0, 0, 2)] + ([(0, 64, 0, 0, 2, 1)] if w.dtype == wl.BF16 else [])
    for tune in tunes:
        out = gh.library_conv3x3(w, vals_lib, X_lib, tune=tune)
        err = orc.normalised_error(out, ref, den)
        print(f"[gpu]   normalised error {err:.3e}", flush=True)
        assert err <= gh.TOL[w.dtype], err


def test_fused_conv3x3_random_geometries():
    """Thirty seeded random (mask, images, height, width, dtype, stage split) combinations."""
    g = np.random.Generator(np.random.PCG64(77))
    shapes = [c[0] for c in CONV_CASES[:3]] + [
        wl.Workload("conv_r6", (2, 3, 4, 2), (2, 2, 4, 9), (1, 2, 2, 9), 0, wl.F32, 81, 82, 83, 1.0),
        wl.Workload("conv_kc18", (4, 2, 4, 2), (4, 1, 4, 9), (2, 1, 2, 9), 0, wl.F32, 84, 85, 86, 1.0),
        wl.Workload("conv_8x8", (8, 2, 4, 1), (8, 2, 4, 9), (2, 2, 2, 9), 0, wl.F32, 87, 88, 89, 1.0)]
    ran = 0
    for it in range(30):
        dtype = int(g.integers(0, 2))
        w = replace(shapes[it % len(shapes)], dtype=dtype, name=f"conv_random{it}")
        B, H, W = int(g.integers(1, 7)), int(g.integers(1, 8)), int(g.choice([4, 8, 12, 16, 20, 32, 64]))
        vals, X = wl.kept_weights(w), wl.conv_activations(w, B, H, W)
        if dtype == wl.BF16:
            vals_lib, X_lib = wl.to_bf16_bits(vals), wl.to_bf16_bits(X)
            vals, X = wl.bf16_bits_as_f32(vals_lib), wl.bf16_bits_as_f32(X_lib)
        else:
            vals_lib, X_lib = vals, X
        out = gh.library_conv3x3(w, vals_lib, X_lib, tune=(0, 0, 0, 0, 0, int(g.choice([0, 1, 2, 4]))))
        ref, den = gh.oracle_spmm(w, vals, orc.im2col_3x3(X))
        err = orc.normalised_error(out, ref, den)
        assert err <= gh.TOL[dtype], (w.rows, B, H, W, dtype, err)
        ran += 1
    assert ran == 30


def test_fused_conv3x3_argument_checks():
    import torch
    w, B, H, W = CONV_CASES[0]
    mask = rb.rbgp_make_mask(w.rows, w.cols, w.row_deg, w.mask_seed)
    buf = torch.zeros(1 << 20, dtype=torch.float32, device="cuda:0")
    args = (buf.data_ptr(), buf.data_ptr(), buf.data_ptr())
    for bad, code in [(dict(width=6), rb.ESHAPE), (dict(cin=w.K // 9 + 1), rb.ESHAPE)]:
        with pytest.raises(rb.RbgpError) as ei:
            rb.rbgp_conv3x3(mask, bad.get("dtype", rb.F32), w.M, bad.get("cin", w.K // 9), B, H, bad.get("width", W),
                            args[0], args[1], args[2], B * H * bad.get("width", W), 0)
        assert ei.value.code == code
    # a mask whose G_b does not have the nine taps
    m2 = rb.rbgp_make_mask(wl.TINY.rows, wl.TINY.cols, wl.TINY.row_deg, 1)
    with pytest.raises(rb.RbgpError):
        rb.rbgp_conv3x3(m2, rb.F32, wl.TINY.M, wl.TINY.K // 9, 1, 4, 4, args[0], args[1], args[2], 16, 0)


def test_masks_outside_rbgp4_roles_use_the_generic_kernel():
    """Sparse G_r / G_b (general four-factor RBGP): the kernels' view folds them into G_o / G_i and the MFMA
    kernels run; more than 16 rows in G_b alone leaves the register family."""
    w = wl.Workload("general_rbgp", (4, 4, 4, 2), (4, 4, 8, 4), (2, 2, 4, 2), 130, wl.F32, 5, 6, 7, 1.0)
    gh.check_parity(w, expect_kernel=REG)
    gh.check_parity(w, kernel=GEN)
    gh.check_parity(replace(w, dtype=wl.BF16), ld_pad=2, expect_kernel=REG)     # (bf16: leading dimension a multiple of 4)
    big_gb = wl.Workload("big_gb", (2, 1, 2, 32), (2, 1, 4, 3), (2, 1, 2, 3), 96, wl.F32, 8, 9, 10, 1.0)
    assert not gh.family_covers(big_gb, REG)
    gh.check_parity(big_gb)


def test_sdmm4096_paper_workload_sampled():
    """Table 2's 4096^3 SDMM at 87.5 % sparsity, (50 %, 75 %) split: full shape
    on the GPU, a sample of output columns checked against the oracle."""
    w = wl.sdmm4096_table2(1, 2)
    vl, Il, vf, If = gh.host_inputs(w)
    cols = np.r_[0:64, 2000:2064, 4032:4096]
    ref, den = gh.oracle_spmm(w, vf, np.ascontiguousarray(If[:, cols]))
    # the default launch (the register family on the mask with G_o filled in and merged with G_r), the register family on
    # the mask as given (stage lists split over the waves of a workgroup) and the LDS family
    for kernel, want in ((rb.KERNEL_AUTO, FILLED), (REG, REG), (MFMA, MFMA), (FILLED, FILLED)):
        out, used = gh.library_spmm(w, vl, Il, kernel=kernel, tag="table2")
        assert used == want
        assert orc.normalised_error(out[:, cols], ref, den) <= gh.TOL[w.dtype]


# ------------------------------------------------------------------ random masks, library defaults
def _random_shapes(count, seed):
    """Seeded random four-factor shapes (G_r, G_b complete) that the sampler accepts."""
    g = np.random.Generator(np.random.PCG64(seed))
    shapes = []
    while len(shapes) < count:
        lo, li = int(g.integers(0, 3)), int(g.integers(0, 3))            # log2 of G_o's / G_i's inverse density
        a_o = int(g.choice([1, 2, 3, 4, 6, 8, 12, 16])) << lo
        c_o = int(g.choice([1, 2, 3, 4, 8])) << lo
        a_i = int(g.choice([1, 2, 4])) << li
        c_i = int(g.choice([1, 2, 4])) << li
        a_r, c_r = int(g.choice([1, 2, 3, 4, 8])), int(g.choice([1, 2, 3, 4]))
        a_b, c_b = int(g.choice([1, 2, 3, 4, 24])), int(g.choice([1, 3, 9, 9]))
        rows, cols = (a_o, a_r, a_i, a_b), (c_o, c_r, c_i, c_b)
        deg = (c_o >> lo, c_r, c_i >> li, c_b)
        if a_o * a_r * a_i * a_b > 2048 or c_o * c_r * c_i * c_b > 4096:
            continue
        try:
            rb.rbgp_make_mask(rows, cols, deg, 900 + len(shapes))
        except rb.RbgpError:
            continue
        shapes.append((rows, cols, deg, int(g.integers(1, 700))))
    return shapes


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
def test_random_masks_with_library_defaults(dtype):
    """Forty seeded random shapes, ragged column counts, whatever kernel and launch shape the
    library chooses for them."""
    used = set()
    for idx, (rows, cols, deg, N) in enumerate(_random_shapes(40, 2024)):
        w = wl.Workload(f"random{idx}_{dtype}", rows, cols, deg, N, dtype, 900 + idx, 1000 + idx, 1100 + idx, 1.0)
        vl, Il, vf, If = gh.host_inputs(w)
        out, kernel = gh.library_spmm(w, vl, Il, ld_pad=(-N) % 8)    # a leading dimension every family accepts
        used.add(kernel)
        ref, den = gh.oracle_spmm(w, vf, If)
        err = orc.normalised_error(out, ref, den)
        assert err <= gh.TOL[dtype], (rows, cols, deg, N, kernel, err)
    assert rb.KERNEL_MFMA_REG in used and len(used) >= 2, used


# ------------------------------------------------------------------ more than four base graphs
K_WORKLOADS = [
    wl.Workload("k6_two_sparse_in_go_taps_3x3", (2, 2, 2, 4, 2, 2), (4, 2, 2, 8, 3, 3), (2, 1, 2, 4, 3, 3), 200, wl.F32,
                91, 92, 93, 1.0, roles=(0, 0, 1, 2, 3, 3)),
    wl.Workload("k5_three_in_gi", (4, 4, 2, 2, 3), (4, 8, 2, 4, 1), (2, 4, 2, 2, 1), 136, wl.F32,
                94, 95, 96, 1.0, roles=(0, 2, 2, 2, 3)),
    wl.Workload("k3_no_gb", (4, 2, 4), (8, 2, 4), (2, 2, 2), 72, wl.F32, 97, 98, 99, 1.0, roles=(0, 1, 2)),
    wl.Workload("k5_sparse_gr", (4, 2, 2, 4, 2), (4, 4, 2, 4, 2), (2, 2, 2, 2, 2), 100, wl.F32,
                100, 101, 102, 1.0, roles=(0, 1, 1, 2, 3)),          # sparse graph given to G_r: regrouped by the library
    wl.Workload("k5_sparse_graph_joins_go", (4, 2, 2, 4, 2), (4, 4, 2, 4, 2), (2, 2, 2, 2, 2), 100, wl.F32,
                100, 101, 102, 1.0, roles=(0, 0, 1, 2, 3)),          # the same graphs, the sparse second one in G_o: MFMA
]


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("w", K_WORKLOADS, ids=lambda w: w.name)
def test_masks_of_more_than_four_base_graphs(w, dtype):
    """Section 5: a mask is configured by the number of base graphs and their types; the library
    folds them into the four factors of its kernels."""
    w = replace(w, dtype=dtype)
    err = gh.check_parity(w)
    assert gh.family_covers(w, REG)
    gh.check_parity(w, kernel=REG, expect_kernel=REG)
    gh.check_parity(w, kernel=GEN)
    # backward products of the same masks
    lib, f32 = gh.backward_inputs(w)
    dI_ref, dI_den, dW_ref, dW_den = gh.oracle_backward(w, *f32)
    dI, _ = gh.library_spmm_transposed(w, lib[0], lib[2])
    assert orc.normalised_error(dI, dI_ref, dI_den) <= gh.TOL[dtype]
    dW = gh.library_sddmm(w, lib[2], lib[1])
    assert orc.normalised_error(dW, dW_ref, dW_den) <= gh.TOL[dtype]


def test_non_finite_input_stays_in_its_column():
    """An infinity in one element of I: on the plain kernel it reaches exactly the rows of W_s that keep a
    weight in that column of the mask (the sum of Section 5 runs over kept weights only); on the MFMA
    families, whose padding multiplies zero weights by real rows of I, it may spoil other rows of the same
    column of O, and never another column."""
    w = replace(wl.VGG19_CONV5, rows=(4, 4, 4, 2), cols=(4, 4, 8, 9), row_deg=(2, 4, 2, 9), name="non_finite")
    N, k_bad, n_bad = 200, 37, 77
    vl, Il, vf, If = gh.host_inputs(w, N)
    I_bad = Il.copy()
    I_bad[k_bad, n_bad] = np.inf
    mask = gh.make_mask(w)
    touched = rb.rbgp_mask_dense(mask).reshape(w.M, w.K)[:, k_bad].astype(bool)
    assert touched.any() and not touched.all()
    for kernel in (GEN, MFMA, REG):
        clean, _ = gh.library_spmm(w, vl, Il, kernel=kernel, tag="finite")
        spoilt, _ = gh.library_spmm(w, vl, I_bad, kernel=kernel, tag="one infinity")
        others = np.ones(N, bool)
        others[n_bad] = False
        assert np.array_equal(clean[:, others].view(np.uint32), spoilt[:, others].view(np.uint32))
        assert not np.isfinite(spoilt[touched, n_bad]).any()
        if kernel == GEN:
            assert np.array_equal(clean[~touched, n_bad].view(np.uint32), spoilt[~touched, n_bad].view(np.uint32))


# masks of 3x3 convolutions whose G_i has groups of vertices with one adjacency list: the register family runs on the mask with a
# group's rows in G_r, rows permuted (rows, cols, degrees, rows per column set before and after)
MERGED_ROW_SHAPES = [
    ((8, 4, 8, 1), (8, 4, 4, 9), (4, 4, 1, 9), 4, 8),     # pairs: tile rows paired tile by tile where the batch fills the chip
    ((6, 2, 8, 1), (4, 2, 2, 9), (2, 2, 1, 9), 2, 8),     # fours, six tile rows
    ((4, 4, 16, 1), (4, 1, 4, 9), (4, 1, 1, 9), 4, 16),   # fours: whole MFMA groups
    ((4, 1, 8, 2), (8, 1, 4, 9), (2, 1, 1, 9), 2, 4),     # rows of G_b next to the merged ones
]


@pytest.mark.parametrize("idx", range(len(MERGED_ROW_SHAPES)))
@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
def test_register_family_on_the_mask_with_merged_rows(idx, dtype):
    rows, cols, deg, before, after = MERGED_ROW_SHAPES[idx]
    w = wl.Workload(f"merged_rows{idx}", rows, cols, deg, 0, dtype, 310 + idx, 320 + idx, 330 + idx, 1.0)
    mask = rb.rbgp_make_mask(rows, cols, deg, w.mask_seed)
    plan = rb.rbgp_mask_reg_plan(mask)
    assert rows[1] * rows[3] == before and plan[14] == after
    rb.rbgp_mask_check_tables(mask)
    for N in (8, 328, 4104):   # split lists, a ragged last tile, whole lists (and pairs of tile rows)
        gh.check_parity(w, N=N, kernel=REG, ld_pad=8, expect_kernel=REG)
    gh.check_parity(w, N=200, kernel=REG, tune=(0, 0, 0, 1, 0, 0), expect_kernel=REG)
    vals, X = wl.kept_weights(w), wl.conv_activations(w, 37, 4, 8)
    if dtype == wl.BF16:
        vals, X = wl.to_bf16_bits(vals), wl.to_bf16_bits(X)
    out = gh.library_conv3x3(w, vals, X)
    as_f32 = wl.bf16_bits_as_f32 if dtype == wl.BF16 else (lambda a: a)
    ref, den = gh.oracle_spmm(w, as_f32(vals), orc.im2col_3x3(as_f32(X)))
    assert orc.normalised_error(out, ref, den) <= gh.TOL[dtype]


@pytest.mark.parametrize("tune,N", [((0,) * 7 + (1,), 4104), ((0,) * 7 + (1,), 64), ((0,) * 7 + (2,), 4104)])
def test_merged_rows_take_the_knobs_of_the_mask_as_given(tune, N):
    """fp32 with four rows per column set: RBGP_TUNE_REGISTER_SETS where the default pairs the merged tile rows, and no
    RBGP_TUNE_ROW_PAIRING = 2, which masks of such rows refuse."""
    rows, cols, deg, *_ = MERGED_ROW_SHAPES[0]
    w = wl.Workload("merged_knobs", rows, cols, deg, N, wl.F32, 310, 320, 330, 1.0)
    gh.check_parity(w, kernel=REG, expect_kernel=REG)
    assert rb.rbgp_last_kernel() == ("spmm_reg_dual" if N > 64 else "spmm_reg_narrow")
    gh.check_parity(w, kernel=REG, tune=tune, expect_kernel=REG)
    assert rb.rbgp_last_kernel() == "spmm_reg"
    with pytest.raises(rb.RbgpError) as e:
        gh.check_parity(w, kernel=REG, tune=(0, 0, 0, 2))
    assert e.value.code == rb.EUNSUPPORTED


# (mask, element type, columns of the eager call, of the captured one): merged rows; tile rows paired without them; bf16 clusters of
# one, two and four groups of rows
OTHER_WIDTHS = [(MERGED_ROW_SHAPES[0][:3], wl.F32, 40960, 64), (MERGED_ROW_SHAPES[0][:3], wl.F32, 64, 40960),
                (MERGED_ROW_SHAPES[1][:3], wl.F32, 40960, 64), (MERGED_ROW_SHAPES[1][:3], wl.BF16, 40960, 64),
                (MERGED_ROW_SHAPES[2][:3], wl.BF16, 40960, 64), (MERGED_ROW_SHAPES[2][:3], wl.BF16, 64, 40960),
                (((16, 4, 4, 2), (16, 4, 8, 9), (8, 4, 2, 9)), wl.F32, 2048, 64), (((16, 4, 4, 2), (16, 4, 8, 9), (8, 4, 2, 9)), wl.F32, 64, 2048),
                (MERGED_ROW_SHAPES[0][:3], wl.BF16, 64, 40960),
                (((32, 4, 32, 4), (16, 1, 32, 1), (8, 1, 16, 1)), wl.BF16, 64, 4096), (((32, 4, 32, 4), (16, 1, 32, 1), (8, 1, 16, 1)), wl.BF16, 4096, 64)]


@pytest.mark.parametrize("mask_of,dtype,first,then", OTHER_WIDTHS)
def test_register_family_on_another_batch_allocates_nothing(mask_of, dtype, first, then):
    """An eager call, then the capture of one on another number of columns, which other kernels and clusters take: three replays
    on fresh inputs against the eager result."""
    import torch
    w = wl.Workload("other_width", *mask_of, 0, dtype, 310, 320, 330, 1.0)
    mask, ld = gh.make_mask(w), max(first, then)
    rb.rbgp_mask_set_kernel(mask, REG)
    t = torch.float32 if dtype == wl.F32 else torch.bfloat16
    stream = lambda: torch.cuda.current_stream().cuda_stream
    packed = torch.zeros(rb.rbgp_packed_bytes(mask, dtype), dtype=torch.uint8, device="cuda:0")
    vals = wl.kept_weights(w)
    rb.rbgp_pack(mask, dtype, wl.to_bf16_bits(vals) if dtype == wl.BF16 else vals, packed.data_ptr(), stream())
    I, O = torch.zeros((w.K, ld), dtype=t, device="cuda:0"), torch.zeros((w.M, ld), device="cuda:0")
    call = lambda n: rb.rbgp_spmm(mask, dtype, w.M, w.K, n, packed.data_ptr(), I.data_ptr(), ld, O.data_ptr(), ld, stream())
    if dtype == wl.BF16 and w.cols[3] == 9 and first > then:   # (a convolution before: it looks at clusters of two groups, too)
        rb.rbgp_conv3x3(mask, dtype, w.M, w.K // 9, 1, 4, 8, packed.data_ptr(), I.data_ptr(), O.data_ptr(), 32, stream())
    call(first)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(then)
    for seed in (1, 2, 3):
        I.copy_(torch.randn(I.shape, device="cuda:0", generator=torch.Generator(device="cuda:0").manual_seed(seed)))
        O.fill_(float("nan"))
        call(then)
        torch.cuda.synchronize()
        want = O[:, :then].clone()
        O.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(O[:, :then], want)
        call(first)


@pytest.mark.parametrize("N", [1, 63, 100, 2047, 2112, 6700])
def test_lds_family_split_operands_by_width(N):
    """Two groups of waves, 64 and 128 columns a workgroup, ragged last tiles; one column that is not finite stays by itself."""
    w = wl.Workload("split_tiles", (8, 4, 32, 1), (32, 1, 32, 1), (8, 1, 8, 1), N, wl.F32, 351, 352, 353, 1.0)
    vl, I, _, _ = gh.host_inputs(w, N)
    I = I.copy()
    I[7, N - 1] = np.inf
    out, used = gh.library_spmm(w, vl, I, kernel=MFMA, ld_pad=(-N) % 4)
    assert used == MFMA and rb.rbgp_last_kernel() == f"spmm_mfma_split<8, 1, {'2, 2' if N < 2112 else '2, 1' if N < 6700 else '4, 1'}>"
    with np.errstate(invalid="ignore"):
        ref, den = gh.oracle_spmm(w, vl, I)
    assert np.array_equal(np.isfinite(out), np.isfinite(ref))
    fin = np.isfinite(ref)
    assert orc.normalised_error(out[fin], ref[fin], den[fin]) <= gh.TOL[wl.F32] / 10   # (split operands: below the fp32 forms' 1e-6)


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("side", [7, 64, 724, 725])
def test_pack_writes_the_layout(side, shift, dtype):
    """One element a thread and four (from 524 288 on, aligned buffers only), with a remainder; nothing past the packed weights."""
    import torch
    mask = rb.rbgp_make_mask((1, side, 1, 1), (1, side, 1, 1), (1, side, 1, 1), 371)   # nnz = side * side
    rb.rbgp_mask_set_kernel(mask, GEN)
    layout = rb.rbgp_pack_layout(mask, dtype)
    vals = torch.randn(side * side, device="cuda:0").to(torch.float32 if dtype == wl.F32 else torch.bfloat16)
    out = torch.full((layout.size + 8,), 3.0, dtype=vals.dtype, device="cuda:0")
    rb.rbgp_pack_device(mask, dtype, vals.data_ptr(), out.data_ptr() + shift * out.element_size(), 0)
    torch.cuda.synchronize()
    want = torch.where(torch.from_numpy(layout < 0), 0.0, vals.float().cpu()[torch.from_numpy(np.maximum(layout, 0)).long()])
    got = out.float().cpu()
    assert torch.equal(got[shift:shift + layout.size], want)
    assert (got[:shift] == 3.0).all() and (got[shift + layout.size:] == 3.0).all()


# VGG19 layers on few columns: workgroups of 16 columns and eight waves a list (layer, log2 of 1 / density, transposed), stages of
# 72 steps in clusters of one, two and four tile rows, of 36, in fp32 of 32 and of 18
NARROW = [(13, 1, False), (13, 2, False), (4, 4, False), (3, 4, False), (13, 1, True), (13, 2, True)]


@pytest.mark.parametrize("N", [1, 15, 17, 64])
@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("layer, density_log2, transposed", NARROW)
def test_register_family_on_few_columns(layer, density_log2, transposed, dtype, N):
    w = replace(wl.vgg19_sweep_workload(layer, density_log2, dtype), N=N)
    if transposed:
        lib, f32 = gh.backward_inputs(w)
        out, used = gh.library_spmm_transposed(w, lib[0], lib[2], ld_pad=(-N) % 8)
        ref, den, _, _ = gh.oracle_backward(w, *f32)
    else:
        vl, I, vals_f, I_f = gh.host_inputs(w, N)
        out, used = gh.library_spmm(w, vl, I, kernel=REG, ld_pad=(-N) % 8 + 8)
        ref, den = gh.oracle_spmm(w, vals_f, I_f)
    assert used == REG
    if dtype == wl.F32:   # (transposes have 288 and 384 lists; the bf16 kernels take 128 columns a wave or share them first)
        assert (rb.rbgp_last_kernel() == "spmm_reg_narrow") == (N <= 16 or not transposed)
    elif not transposed:
        assert rb.rbgp_last_kernel() == "spmm_reg_narrow"
    assert orc.normalised_error(out, ref, den) <= gh.TOL[dtype]


# stages of 18 and 32 steps with few lists (bf16: one group of rows on 64 columns), and lists of up to 128 stages
NARROW_MASKS = [((4, 4, 4, 2), (4, 1, 4, 9), (2, 1, 2, 9)), ((4, 4, 8, 2), (4, 1, 64, 1), (2, 1, 32, 1)), ((2, 4, 4, 2), (128, 1, 4, 9), (64, 1, 2, 9))]


@pytest.mark.parametrize("N", [1, 17, 63])
@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("rows,cols,deg", NARROW_MASKS)
def test_few_columns_on_short_stages_and_long_lists(rows, cols, deg, dtype, N):
    w = wl.Workload("narrow", rows, cols, deg, N, dtype, 361, 362, 363, 1.0)
    plan = rb.rbgp_mask_reg_plan(gh.make_mask(w))
    assert plan[2] == (32 if cols[3] == 1 else 18) and (plan[5] > 64) == (cols[0] == 128)
    gh.check_parity(w, kernel=REG, ld_pad=(-N) % 4, expect_kernel=REG)
    assert rb.rbgp_last_kernel() == "spmm_reg_narrow"


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("layer, images", [(9, 1), (9, 3), (4, 1), (13, 5)])
def test_fused_convolution_on_few_columns(layer, images, dtype):
    w = wl.vgg19_sweep_workload(layer, 1, dtype)
    vals, X = wl.kept_weights(w), wl.conv_activations(w, images, 4, 4 if layer != 4 else 8)
    as_f32 = wl.bf16_bits_as_f32 if dtype == wl.BF16 else (lambda a: a)
    if dtype == wl.BF16:
        vals, X = wl.to_bf16_bits(vals), wl.to_bf16_bits(X)
    out = gh.library_conv3x3(w, vals, X)
    assert rb.rbgp_last_kernel() == "spmm_reg_narrow"
    ref, den = gh.oracle_spmm(w, as_f32(vals), orc.im2col_3x3(as_f32(X)))
    assert orc.normalised_error(out, ref, den) <= gh.TOL[dtype]
