"""Which kernels a product of open tile runs on, on both sides of each
line: short loops over several rounds of tiles on the larger tile, long loops
in little more than one round, three products without a probe and int32 on the
packed path where it is the faster one; and the results there, against the oracle or float64.  (The lines depend on the number of
compute units; the sizes are those of 256.)"""
import numpy as np
import pytest

import oracle
import synth
from _util import FP32_REL_FRO_TOL, SEED, rel_fro

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ax():
    import torch

    import paper_1412_1127_amd as ax
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("sizes for 256 compute units")
    ax.acc_init(0, 0)
    yield ax
    ax.acc_shutdown()


def _flags(ax, prec):
    return ax.ACC_KERNEL_TILED | {"auto": ax.ACC_PREC_AUTO, "full6": ax.ACC_PREC_FULL6, "five": ax.ACC_PREC_FIVE,
                                  "cheap3": ax.ACC_PREC_CHEAP3}[prec]


# short loops: 64 x 64 tiles in several rounds pay a round trip to memory (and
# a probe) per round; the probe records show the tile that ran
@pytest.mark.parametrize("m,n,k,edge", [(1000, 1000, 16, 64), (1030, 1030, 16, 128), (2048, 2048, 32, 128),
                                        (3000, 3000, 32, 128), (2200, 2200, 130, 128), (2500, 2500, 64, 128),
                                        (9000, 500, 33, 128), (1000, 1000, 1000, 64)])
def test_tile_of_short_loops(ax, m, n, k, edge):
    import torch
    fl = _flags(ax, "auto")
    off, cnt = ax.accx_gemm_probe_layout(m, n, k, fl)
    assert cnt == -(-m // edge) * -(-n // edge)
    a, b = synth.uniform_pm1_f32((m, k), SEED, 9500), synth.uniform_pm1_f32((k, n), SEED, 9501)
    da, db, dc = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda(), torch.full((m, n), float("nan"), device="cuda")
    ws = ax.accx_gemm_workspace_size(ax.ACC_FLOAT32, m, n, k, fl)
    work = torch.full((ws,), 0xFF, dtype=torch.uint8, device="cuda")
    print("short loop m=%d n=%d k=%d" % (m, n, k), flush=True)
    ax.accx_gemm_dev(ax.ACC_FLOAT32, m, n, k, da, k, db, n, dc, n, fl, work, ws)
    torch.cuda.synchronize()
    assert rel_fro(dc.cpu().numpy(), oracle.gemm(a, b)) <= FP32_REL_FRO_TOL
    recs = ax.probe_records(work[off:off + cnt * 608].cpu().numpy().tobytes(), cnt)
    # every record was written, its samples inside its tile
    nt = -(-n // edge)
    for q, r in enumerate(recs):
        assert q // nt * edge <= min(r.rows) and max(r.rows) < min(m, (q // nt + 1) * edge)
        assert q % nt * edge <= min(r.cols) and max(r.cols) < min(n, (q % nt + 1) * edge)


@pytest.mark.parametrize("prec,m,n,k,direct", [
    ("cheap3", 2048, 2048, 64, True), ("cheap3", 2060, 2060, 64, False), ("cheap3", 2060, 2060, 600, False),
    ("cheap3", 2700, 2700, 1100, False), ("cheap3", 2950, 2950, 1100, True), ("cheap3", 3000, 3000, 64, False),
    ("auto", 2048, 2048, 1700, True), ("auto", 2060, 2060, 1600, True), ("auto", 2060, 2060, 1601, False),
    ("auto", 2400, 2400, 1700, False), ("auto", 2440, 2440, 1700, True),
    ("five", 2048, 2048, 128, True), ("five", 2060, 2060, 128, False), ("full6", 1030, 1030, 800, True), ("full6", 2048, 2048, 128, True),
    ("full6", 2060, 2060, 128, False)])
def test_route(ax, prec, m, n, k, direct):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    da = torch.rand((m, k), generator=g, device="cuda") * 2 - 1
    db = torch.rand((k, n), generator=g, device="cuda") * 2 - 1
    dc = torch.full((m, n), float("nan"), device="cuda")
    print("route %s m=%d n=%d k=%d" % (prec, m, n, k), flush=True)
    ax.accx_timing_enable(True)
    ax.accx_timing_read(reset=True)
    ax.accx_gemm_dev(ax.ACC_FLOAT32, m, n, k, da, k, db, n, dc, n, _flags(ax, prec))
    torch.cuda.synchronize()
    names = set(ax.accx_timing_read(reset=True))
    ax.accx_timing_enable(False)
    if prec == "auto":
        assert ("gemm_direct_auto" in names) == direct and ("pack_bf16x3" in names) != direct, names
    else:
        assert names == ({"gemm_direct"} if direct else {"pack_bf16x3", "gemm_bf16x3"}), names
    ref = da.double() @ db.double()
    err = float((dc.double() - ref).norm() / ref.norm())
    assert err <= FP32_REL_FRO_TOL, err


@pytest.mark.parametrize("m,n,k,direct", [
    (1000, 1000, 1000, True), (1300, 1300, 1300, False), (2048, 2048, 256, True), (2048, 2048, 512, False),
    (1664, 2096, 652, False), (3372, 607, 469, False), (3372, 608, 200, True), (64, 64, 4096, True),
    (130, 75, 4200, True), (128, 128, 8192, True), (300, 1000, 4000, True)])
def test_route_i32(ax, m, n, k, direct):
    # the direct path where it is the faster one on one-digit values
    import torch
    a, b = synth.int_uniform_i32((m, k), -16, 16, SEED, 9520), synth.int_uniform_i32((k, n), -16, 16, SEED, 9521)
    da, db = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    dc = torch.full((m, n), 77, dtype=torch.int32, device="cuda")
    print("route i32 m=%d n=%d k=%d" % (m, n, k), flush=True)
    ax.accx_timing_enable(True)
    ax.accx_timing_read(reset=True)
    ax.accx_gemm_dev(ax.ACC_INT32, m, n, k, da, k, db, n, dc, n, ax.ACC_KERNEL_TILED)
    torch.cuda.synchronize()
    names = set(ax.accx_timing_read(reset=True))
    ax.accx_timing_enable(False)
    assert ("gemm_i8_direct" in names) == direct and ("pack_i8" in names) != direct, names
    assert np.array_equal(dc.cpu().numpy(), oracle.gemm(a, b))


@pytest.mark.parametrize("dtype", ["f32", "i32"])
@pytest.mark.parametrize("m,n,k,parts", [(1030, 1030, 1030, True), (1100, 1100, 1100, True), (1030, 1030, 500, False),
                                         (300, 260, 1200, True)])
def test_k_parts_that_fit_the_workspace(ax, dtype, m, n, k, parts):
    # an estimate that asks for more K parts than the workspace holds would
    # run unsplit; parts leave their sums in the workspace, and nothing else
    # on this path writes there (six products have no probe records)
    import torch
    if dtype == "i32":
        if m > 1000:
            pytest.skip("int32 products of this size run packed")
        a, b = synth.int_uniform_i32((m, k), -16, 16, SEED, 9510), synth.int_uniform_i32((k, n), -16, 16, SEED, 9511)
        t, fl = ax.ACC_INT32, ax.ACC_KERNEL_TILED
    else:
        a, b = synth.uniform_pm1_f32((m, k), SEED, 9510), synth.uniform_pm1_f32((k, n), SEED, 9511)
        t, fl = ax.ACC_FLOAT32, _flags(ax, "full6")
    da, db = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    dc = torch.zeros((m, n), dtype=da.dtype, device="cuda")
    ws = ax.accx_gemm_workspace_size(t, m, n, k, fl)
    work = torch.full((ws + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    print("parts %s m=%d n=%d k=%d" % (dtype, m, n, k), flush=True)
    ax.accx_timing_enable(True)
    ax.accx_timing_read(reset=True)
    ax.accx_gemm_dev(t, m, n, k, da, k, db, n, dc, n, fl, work, ws)
    torch.cuda.synchronize()
    names = set(ax.accx_timing_read(reset=True))
    ax.accx_timing_enable(False)
    assert names == {"gemm_i8_direct" if dtype == "i32" else "gemm_direct"}, names
    assert bool((work[:ws] != 0xA5).any().item()) == parts
    assert bool((work[ws:] == 0xA5).all().item())
    ref = oracle.gemm(a, b)
    c = dc.cpu().numpy()
    assert np.array_equal(c, ref) if dtype == "i32" else rel_fro(c, ref) <= FP32_REL_FRO_TOL
