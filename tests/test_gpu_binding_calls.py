"""The six calls of a step through ctypes and without it: the same launches, the same results bit for bit."""
import pytest
import torch

from paper_2006_13486_amd import binding as rb
from paper_2006_13486_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [rb.F32, rb.BF16_F32ACC])
@pytest.mark.parametrize("stream", [False, True])
def test_same_results_through_ctypes(dtype, stream):
    assert rb._call is not None, "csrc/rbgp_call.c is not built"
    w, images, side = wl.VGG19_CONV3_BF16, 5, 8
    N, C = images * side * side, w.K // 9
    t = torch.float32 if dtype == rb.F32 else torch.bfloat16
    print(f"[gpu] binding calls {w.name} dtype={dtype} stream={stream}", flush=True)
    mask = rb.rbgp_make_mask(w.rows, w.cols, w.row_deg, w.mask_seed)
    mask_t = rb.rbgp_mask_conv3x3_transpose(mask)
    gen = torch.Generator(device="cuda").manual_seed(4)
    normal = lambda *size: torch.randn(size, generator=gen, device="cuda").to(t)
    weights, I, dO, X = normal(w.nnz), normal(w.K, N), normal(w.M, N), normal(C, images, side + 2, side + 2)
    dOp = normal(w.M, images, side + 2, side + 2)
    on = torch.cuda.Stream() if stream else torch.cuda.current_stream()
    tail = (on.cuda_stream,) if stream else ()   # (without: the default stream)
    torch.cuda.synchronize()

    def results(f):
        with torch.cuda.stream(on):
            new = lambda *size: torch.full(size, float("nan"), device="cuda")
            packed, packed_t = (torch.zeros(rb.rbgp_packed_bytes(m, dtype), dtype=torch.uint8, device="cuda") for m in (mask, mask_t))
            O, Oc, dX, dW, dWc = new(w.M, N), new(w.M, N), new(C, N), new(w.nnz), new(w.nnz)
        on.synchronize()
        names = []
        for name, args in [("rbgp_pack_device", (mask, dtype, weights.data_ptr(), packed.data_ptr())),
                           ("rbgp_pack_transposed_device", (mask_t, dtype, weights.data_ptr(), packed_t.data_ptr())),
                           ("rbgp_spmm", (mask, dtype, w.M, w.K, N, packed.data_ptr(), I.data_ptr(), N, O.data_ptr(), N)),
                           ("rbgp_conv3x3", (mask, dtype, w.M, C, images, side, side, packed.data_ptr(), X.data_ptr(), Oc.data_ptr(), N)),
                           ("rbgp_conv3x3", (mask_t, dtype, C, w.M, images, side, side, packed_t.data_ptr(), dOp.data_ptr(), dX.data_ptr(), N)),
                           ("rbgp_sddmm", (mask, dtype, w.M, w.K, N, dO.data_ptr(), N, I.data_ptr(), N, dW.data_ptr())),
                           ("rbgp_conv3x3_sddmm", (mask, dtype, w.M, C, images, side, side, dO.data_ptr(), N, X.data_ptr(), dWc.data_ptr()))]:
            assert f(name)(*args, *tail) is None
            if "pack" not in name:
                names.append(rb.rbgp_last_kernel())
        torch.cuda.synchronize()
        return names, (packed, packed_t, O, Oc, dX, dW, dWc)

    names, fast = results(lambda name: getattr(rb, name))
    names_slow, slow = results(lambda name: rb._WITH_CTYPES[name])
    assert names == names_slow
    for a, b in zip(fast, slow):
        assert torch.equal(a, b) and bool(torch.isfinite(a.float()).all())
