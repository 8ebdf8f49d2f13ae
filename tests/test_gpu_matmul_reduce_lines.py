"""A matmul and a sum in one region on both sides of the lines between the
direct path, the packed path and the co-scheduled pass: the sum is written on
each of them, and the matrix is that of the matmul alone.  (Untuned, on 256 compute
units: 640 tiles of 128 x 128 up to 3200, 256 of 256 x 256 from 3841 on.)"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["auto", "cheap3"])
@pytest.mark.parametrize("length", [1000, 3200, 3201, 3840, 3841])
def test_sum_is_written(prec, length):
    import torch

    import paper_1412_1127_amd as ax
    ax.acc_init(0, 0)
    flags = ax.ACC_KERNEL_TILED | (ax.ACC_PREC_AUTO if prec == "auto" else ax.ACC_PREC_CHEAP3)
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    a, b = [torch.rand((length, length), generator=g, device="cuda") * 2 - 1 for _ in range(2)]
    n = 3000001
    x = torch.rand(n, generator=g, device="cuda")
    c, alone = torch.full_like(a, float("nan")), torch.full_like(a, float("nan"))
    res = torch.full((1,), float("nan"), device="cuda")
    print("matmul+reduce lines len=%d %s" % (length, prec), flush=True)
    names = []
    ax.accx_timing_enable(True)
    for call in (lambda: ax.accx_matmul_reduce_dev(a, b, c, length, flags, x, n, 0.25, res),
                 lambda: ax.accx_matmul_dev(ax.ACC_FLOAT32, a, b, alone, length, flags)):
        ax.accx_timing_read(reset=True)
        call()
        torch.cuda.synchronize()
        names.append(set(ax.accx_timing_read(reset=True)))
    ax.accx_timing_enable(False)
    want = float(x.sum(dtype=torch.float64)) + 0.25
    assert abs(float(res) - want) <= 1e-5 * want
    assert torch.equal(c, alone) and bool(torch.isfinite(c).all())
    # the matmul's own kernels, and a direct one carries no sum
    assert names[1] <= names[0] and names[0] - names[1] <= {"reduce_fast", "reduce_final"}, names
    if names[1] & {"gemm_direct", "gemm_direct_auto"}:
        assert "reduce_fast" in names[0]
    ax.acc_shutdown()
