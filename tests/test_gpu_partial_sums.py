"""Partial sums of the weight gradient, from none to 128 a value, against the product in 64 bits."""
import pytest
import torch

from paper_2006_13486_amd import binding as rb
from paper_2006_13486_amd import workloads as wl
from tests.test_dispatch import FEW_UNITS, PARTIAL_SUMS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [rb.F32, rb.BF16_F32ACC])
@pytest.mark.parametrize("N", [8192, 16384, 24584, 40960, 65536, 131072])
@pytest.mark.parametrize("w", [wl.WRN_G1, wl.vgg19_sweep_workload(1, 1, wl.F32)], ids=lambda w: w.name)
def test_partial_sums(w, N, dtype):
    check(w, N, dtype)


# the counts around those where other kernels add the partial sums, and the most that a mask of two units takes (fp32: 7, 8, 28, 29, 31, 32,
# 113, 118 and 128 a value; test_dispatch.py names the kernels; bf16: up to 128)
@pytest.mark.parametrize("dtype", [rb.F32, rb.BF16_F32ACC])
@pytest.mark.parametrize("k,N", [(k, N) for k, N, _ in PARTIAL_SUMS])
def test_partial_sums_of_few_units(k, N, dtype):
    check(wl.Workload("few_units", *FEW_UNITS[k], 0, dtype, 101, 102, 103, 1.0), N, dtype)


def check(w, N, dtype):
    t_in = torch.float32 if dtype == rb.F32 else torch.bfloat16
    print(f"[gpu] partial sums {w.name} N={N} dtype={dtype}", flush=True)
    mask = rb.rbgp_make_mask(w.rows, w.cols, w.row_deg, w.mask_seed)
    gen = torch.Generator(device="cuda").manual_seed(3)
    dO = torch.randn((w.M, N), generator=gen, device="cuda").to(t_in)
    I = torch.randn((w.K, N), generator=gen, device="cuda").to(t_in)
    dW = torch.full((w.nnz,), float("nan"), device="cuda")
    rb.rbgp_sddmm(mask, dtype, w.M, w.K, N, dO.data_ptr(), N, I.data_ptr(), N, dW.data_ptr())
    torch.cuda.synchronize()
    columns = torch.from_numpy(rb.rbgp_mask_columns(mask)).long().cuda()
    want = torch.zeros((w.M, w.K), dtype=torch.float64, device="cuda")
    for n in range(0, N, 16384):
        want += dO[:, n:n + 16384].double() @ I[:, n:n + 16384].double().T
    want = want.gather(1, columns).reshape(-1)
    # up to 131072 signed products: 2^-24 of a sum's size at each of at most some 1000 additions in a row of a wave's part, whatever the
    # number of parts (512 waves at the most, 256 columns each), 2^-24 sqrt(1000) = 2e-6
    assert (dW.double() - want).norm() <= 2e-6 * want.norm()
