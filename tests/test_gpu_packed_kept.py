"""The packed path at sizes whose open-tile calls run the direct kernels: with a
tile forced, the digit count is still decided from the recorded maxima, the
probe still reads the packed operands, and the workspace may hold anything."""
import numpy as np
import pytest

import oracle
import synth
from _util import FP32_REL_FRO_TOL, SEED, rel_fro
from test_gpu_probe import _biased_split, _check_records

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ax():
    import paper_1412_1127_amd as ax
    ax.acc_init(0, 0)
    yield ax
    ax.acc_shutdown()


def _named(ax, call):
    import torch
    ax.accx_timing_enable(True)
    ax.accx_timing_read(reset=True)
    call()
    torch.cuda.synchronize()
    names = set(ax.accx_timing_read(reset=True))
    ax.accx_timing_enable(False)
    return names


# one element at each side of each digit count's range, as the open-tile test
@pytest.mark.parametrize("tile", ["64", "128", "256"])
@pytest.mark.parametrize("where", ["a", "b"])
def test_i32_digit_count_thresholds(ax, where, tile):
    import torch
    n = 130
    a0 = synth.int_uniform_i32((n, n), -100, 100, SEED, synth.STREAM_A)
    b0 = synth.int_uniform_i32((n, n), -100, 100, SEED, synth.STREAM_B)
    nbytes = ax.accx_matmul_workspace_size(ax.ACC_INT32, n, ax.ACC_KERNEL_TILED | ax.TILES[tile])
    w = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")
    for v in (127, -127, 128, -128, 32639, 32640, -32896, -32897, 8355711, 8355712, -8421504, -8421505, 2 ** 31 - 1,
              -(2 ** 31)):
        a, b = a0.copy(), b0.copy()
        (a if where == "a" else b)[n - 1, 57] = v
        da, db = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
        dc = torch.full((n, n), -7, dtype=torch.int32, device="cuda")
        print("packed thresholds tile=%s %s=%d" % (tile, where, v), flush=True)
        names = _named(ax, lambda: ax.accx_matmul_dev(ax.ACC_INT32, da, db, dc, n, ax.ACC_KERNEL_TILED | ax.TILES[tile],
                                                      w, nbytes))
        assert "pack_i8" in names and "gemm_i8_direct" not in names, names
        assert np.array_equal(dc.cpu().numpy(), oracle.matmul_i32(a, b)), v


@pytest.mark.parametrize("tile", ["128", "256"])
def test_i32_digit_decision_with_reused_and_garbage_workspace(ax, tile):
    import torch
    n = 300
    flags = ax.ACC_KERNEL_TILED | ax.TILES[tile]
    small = [synth.int_uniform_i32((n, n), -100, 100, SEED, 61 + k) for k in range(2)]
    big = [synth.full_range_i32((n, n), SEED, 63 + k) for k in range(2)]
    mid = [synth.int_uniform_i32((n, n), -30000, 30000, SEED, 65 + k) for k in range(2)]
    nbytes = ax.accx_matmul_workspace_size(ax.ACC_INT32, n, flags)
    w = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")
    g = synth.rng(SEED, 67)
    for k, (a, b) in enumerate([small, big, small, mid, small, big, [small[0], big[1]], [mid[0], small[1]]]):
        if k in (4, 6):
            w.copy_(torch.from_numpy(g.integers(0, 256, nbytes).astype(np.uint8)).cuda())
        da, db = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
        dc = torch.full((n, n), -7, dtype=torch.int32, device="cuda")
        print("packed int32 with a reused workspace tile=%s call %d" % (tile, k), flush=True)
        ax.accx_matmul_dev(ax.ACC_INT32, da, db, dc, n, flags, w, nbytes)
        torch.cuda.synchronize()
        assert np.array_equal(dc.cpu().numpy(), oracle.matmul_i32(a, b)), k


@pytest.mark.parametrize("tile", ["64", "128", "256x128", "256"])
@pytest.mark.parametrize("n,biased", [(100, False), (257, False), (1000, False), (256, True), (300, True)])
def test_probe_records(ax, n, biased, tile):
    import torch
    if biased:
        g = synth.rng(SEED, 8)
        a, b = _biased_split(g, (n, n)), _biased_split(g, (n, n))
    else:
        a = synth.uniform_pm1_f32((n, n), SEED, synth.STREAM_A)
        b = synth.uniform_pm1_f32((n, n), SEED, synth.STREAM_B)
    flags = ax.ACC_KERNEL_TILED | ax.ACC_PREC_AUTO | ax.TILES[tile]
    ws = torch.full((ax.accx_matmul_workspace_size(ax.ACC_FLOAT32, n, flags),), 0xFF, dtype=torch.uint8, device="cuda")
    da, db = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    dc, dcc = torch.empty((n, n), device="cuda"), torch.empty((n, n), device="cuda")
    print("packed probe LEN=%d tile=%s biased=%d" % (n, tile, biased), flush=True)
    names = _named(ax, lambda: ax.accx_matmul_dev(ax.ACC_FLOAT32, da, db, dc, n, flags, ws, ws.numel()))
    assert {"pack_bf16x3", "gemm_bf16x3", "probe_f64"} <= names, names
    ax.accx_matmul_dev(ax.ACC_FLOAT32, da, db, dcc, n, ax.ACC_KERNEL_TILED | ax.ACC_PREC_CHEAP3 | ax.TILES[tile])
    torch.cuda.synchronize()
    off, cnt = ax.accx_probe_layout(n, flags)
    recs = ax.probe_records(ws.cpu().numpy().tobytes()[off:], cnt)
    c, cheap = dc.cpu().numpy(), dcc.cpu().numpy()
    _check_records(a, b, cheap, recs)
    assert rel_fro(c, oracle.matmul_f32(a, b)) <= FP32_REL_FRO_TOL
    if biased:
        assert all(r.corrected for r in recs)
