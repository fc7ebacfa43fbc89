"""Rows of O that begin at any element: their stores stay inside the row, and the sums are those of aligned rows."""
import pytest
import torch

from paper_2006_13486_amd import binding as rb
from paper_2006_13486_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [  # (workload, columns, transposed, dtype, kernel)
    (wl.VGG19_CONV5, 2045, False, rb.F32, "spmm_reg_dual"),
    (wl.VGG19_CONV5, 1021, False, rb.F32, "spmm_reg"),
    (wl.VGG19_CONV3_BF16, 8189, False, rb.BF16_F32ACC, "spmm_reg_bf16"),
    (wl.VGG19_CONV3_BF16, 8189, False, rb.BF16, "spmm_reg_bf16"),
    (wl.VGG19_CONV3_BF16, 1023, False, rb.BF16, "spmm_reg_bf16"),
    (wl.sdmm4096_table3(2, 2, 3), 3999, False, rb.BF16_F32ACC, "spmm_reg_bf16_shared<2, 2>"),
    (wl.sdmm4096_table3(2, 2, 3), 3999, False, rb.BF16, "spmm_reg_bf16_shared<2, 2>"),
    (wl.sdmm4096_table3(1, 2, 3), 3374, False, rb.BF16, "spmm_reg_bf16_shared<1, 2>"),
    (wl.sdmm4096_table3(1, 1, 3), 1501, False, rb.F32, "spmm_reg_split"),
    (wl.vgg19_sweep_workload(6, 2, wl.F32), 2369, True, rb.F32, "spmm_reg_rows<3>"),
    (wl.vgg19_sweep_workload(6, 2, wl.F32), 8191, True, rb.F32, "spmm_reg_rows<2>"),
    (wl.vgg19_sweep_workload(6, 2, wl.F32), 2361, True, rb.F32, "spmm_reg_rows<3>"),
    (wl.WRN_G1, 45001, True, rb.F32, "spmm_reg"),              # (99 MB of O: through the caches, several column tiles a wave)
    (wl.vgg19_sweep_workload(1, 2, wl.F32), 47003, True, rb.F32, "spmm_reg"),
]


@pytest.mark.parametrize("shift", [0, 1, 3])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0].name}_{c[1]}_{c[3]}")
def test_rows_that_begin_at_any_element(case, shift):
    w, N, transposed, dtype, kernel = case
    t_in = torch.float32 if dtype == rb.F32 else torch.bfloat16
    t_out = torch.bfloat16 if dtype == rb.BF16 else torch.float32
    print(f"[gpu] unaligned rows {w.name} N={N} dtype={dtype} shift={shift}", flush=True)
    mask = rb.rbgp_make_mask(w.rows, w.cols, w.row_deg, w.mask_seed)
    M, K = w.M, w.K
    gen = torch.Generator(device="cuda").manual_seed(7)
    weights = (torch.randn(w.nnz, generator=gen, device="cuda") * w.w_std).to(t_in)
    if transposed:
        mask, M, K = rb.rbgp_mask_transpose(mask), K, M
    packed = torch.zeros(rb.rbgp_packed_bytes(mask, dtype), dtype=torch.uint8, device="cuda")
    pack = rb.rbgp_pack_transposed_device if transposed else rb.rbgp_pack_device
    pack(mask, dtype, weights.data_ptr(), packed.data_ptr())
    ldI = -(-N // 8) * 8
    I = torch.randn((K, ldI), generator=gen, device="cuda").to(t_in)

    def product(ldO, first):
        out = torch.full((M * ldO + first + 8,), -77.0, dtype=t_out, device="cuda")
        rb.rbgp_spmm(mask, dtype, M, K, N, packed.data_ptr(), I.data_ptr(), ldI, out.data_ptr() + first * out.element_size(), ldO)
        torch.cuda.synchronize()
        rows = out[first:first + M * ldO].view(M, ldO)
        assert (out[:first] == -77).all() and (out[first + M * ldO:] == -77).all() and (rows[:, N:] == -77).all()
        return rows[:, :N].float()

    got = product(N + (N % 2 == 0), shift)   # (an odd leading dimension)
    assert rb.rbgp_last_kernel().split(" +")[0].startswith(kernel), rb.rbgp_last_kernel()
    want = product(-(-N // 8) * 8, 0)
    # The dispatch may take another kernel for aligned rows: another order of at most 1152 fp32 sums (2^-24 sqrt(1152) = 2e-6 of the
    # result's norm), and where O is bf16 a rounding that falls the other way (2^-9 of a value, in few of them).
    assert (got - want).norm() <= (2e-3 if dtype == rb.BF16 else 2e-6) * want.norm()


@pytest.mark.parametrize("layer,ldO,kernel", [(3, 3728269, "spmm_reg_rows<2>"), (3, 3728270, "spmm_reg_rows<2, 1>"), (6, 3728269, "spmm_reg_rows<3>"),
                                              (6, 3728271, "spmm_reg_rows<3, 1>"), (3, 5000001, "spmm_reg_rows<2, 1>")])
def test_rows_of_o_up_to_4_gib_of_a_workgroup_and_beyond(layer, ldO, kernel):
    """The last leading dimension at which a workgroup's 288 rows of O lie within 32-bit offsets, the first ones beyond: the same sums."""
    w, N = wl.vgg19_sweep_workload(layer, 2, wl.F32), 2999
    print(f"[gpu] far rows of O {w.name} ldO={ldO}", flush=True)
    mask = rb.rbgp_mask_transpose(rb.rbgp_make_mask(w.rows, w.cols, w.row_deg, w.mask_seed))
    gen = torch.Generator(device="cuda").manual_seed(8)
    weights = torch.randn(w.nnz, generator=gen, device="cuda") * w.w_std
    packed = torch.zeros(rb.rbgp_packed_bytes(mask, rb.F32), dtype=torch.uint8, device="cuda")
    rb.rbgp_pack_transposed_device(mask, rb.F32, weights.data_ptr(), packed.data_ptr())
    dO = torch.randn((w.M, 3000), generator=gen, device="cuda")

    def product(ld):
        out = torch.full((w.K, ld), -77.0, device="cuda")
        rb.rbgp_spmm(mask, rb.F32, w.K, w.M, N, packed.data_ptr(), dO.data_ptr(), 3000, out.data_ptr(), ld)
        torch.cuda.synchronize()
        assert bool((out[:, N:] == -77).all())
        return out[:, :N].clone()

    near = product(3000)
    assert rb.rbgp_last_kernel() == kernel.replace(", 1>", ">")
    far = product(ldO)
    assert rb.rbgp_last_kernel() == kernel
    assert torch.equal(far, near)
