"""The direct kernels on 128 x 128 tiles, where only larger results take them:
ragged rows, columns and K tails, one and several K parts, every precision and
digit count, rows of any alignment, digit counts that change along K, marked
tiles, infinities and NaN, against the oracle.  (The tile that a shape takes:
for 256 compute units; AUTO's probe records show it.)"""
import numpy as np
import pytest

import oracle
import synth
from _util import FP32_REL_FRO_TOL, SEED, rel_fro
from test_gpu_gemm_direct import CHEAP_REL, _flags, _run
from test_gpu_i8_direct import _run as _run_i8, _values

pytestmark = pytest.mark.gpu

# a K loop of one stage and a tail, of a few, of many; two and three K parts
SHAPES = [(1409, 1537, 33), (2047, 1921, 97), (1409, 1537, 300), (1537, 1409, 531), (1030, 1100, 1040),
          (900, 1100, 1700)]


@pytest.fixture(scope="module")
def ax():
    import torch

    import paper_1412_1127_amd as ax
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("shapes for 256 compute units")
    ax.acc_init(0, 0)
    yield ax
    ax.acc_shutdown()


def _tiles128(m, n):
    return -(-m // 128) * -(-n // 128)


@pytest.mark.parametrize("prec", ["auto", "full6", "five", "cheap3"])
@pytest.mark.parametrize("m,n,k", SHAPES)
def test_f32(ax, m, n, k, prec):
    a, b = synth.uniform_pm1_f32((m, k), SEED, 9700), synth.uniform_pm1_f32((k, n), SEED, 9701)
    if prec == "auto":
        assert ax.accx_gemm_probe_layout(m, n, k, _flags(ax, prec))[1] == _tiles128(m, n)
    c, names = _run(ax, a, b, _flags(ax, prec))
    assert names == {"gemm_direct_auto" if prec == "auto" else "gemm_direct"}, names
    ref = oracle.gemm(a, b)
    if prec in ("five", "cheap3"):
        scale = np.abs(a).astype(np.float64) @ np.abs(b).astype(np.float64)
        assert np.all(np.abs(c - ref) <= (CHEAP_REL + k * 2.0 ** -23) * scale + 1e-30)
    else:
        assert rel_fro(c, ref) <= FP32_REL_FRO_TOL
    for pad, offset in [((3, 1), (1, 3)), ((4, 8), (2, 0))]:
        assert np.array_equal(_run(ax, a, b, _flags(ax, prec), pad, offset)[0], c)


@pytest.mark.parametrize("m,n,k", [(1409, 1537, 33), (1409, 1537, 300), (1030, 1100, 1040)])
def test_marked_tiles(ax, m, n, k):
    import torch
    g = synth.rng(SEED, 98)

    def biased(shape):
        h = 1.0 + g.integers(0, 16, shape) * 2.0 ** -7
        mid = 2.0 ** -9 * (1.0 + g.integers(64, 128, shape) * 2.0 ** -7)
        lo = 2.0 ** -18 * (1.0 + g.integers(16, 32, shape) * 2.0 ** -5)
        return (h + mid + lo).astype(np.float32)

    a, b = biased((m, k)), biased((k, n))
    ref = oracle.gemm(a, b)
    fl = _flags(ax, "auto")
    ws = ax.accx_gemm_workspace_size(ax.ACC_FLOAT32, m, n, k, fl)
    off, cnt = ax.accx_gemm_probe_layout(m, n, k, fl)
    assert cnt == _tiles128(m, n)
    da, db = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    dc = torch.full((m, n), float("nan"), device="cuda")
    work = torch.full((ws,), 0xFF, dtype=torch.uint8, device="cuda")
    print("direct 128 marked m=%d n=%d k=%d" % (m, n, k), flush=True)
    ax.accx_gemm_dev(ax.ACC_FLOAT32, m, n, k, da, k, db, n, dc, n, fl, work, ws)
    torch.cuda.synchronize()
    assert rel_fro(dc.cpu().numpy(), ref) <= FP32_REL_FRO_TOL
    recs = ax.probe_records(work[off:off + cnt * 608].cpu().numpy().tobytes(), cnt)
    assert all(r.corrected == 1 for r in recs)


@pytest.mark.parametrize("prec", ["auto", "full6"])
@pytest.mark.parametrize("m,n,k", [(130, 130, 130), (1409, 1537, 97)])
def test_infinities_and_nan(ax, m, n, k, prec):
    # an infinity or NaN reaches the same entries as on the packed path, and a
    # probe that samples one decides and ends like any other
    a, b = synth.uniform_pm1_f32((m, k), SEED, 9710), synth.uniform_pm1_f32((k, n), SEED, 9711)
    a[3, 7] = np.inf
    a[70, k - 1] = np.nan
    b[k - 1, 5] = -np.inf
    c, names = _run(ax, a, b, _flags(ax, prec))
    assert names == {"gemm_direct_auto" if prec == "auto" else "gemm_direct"}, names
    forced, _ = _run(ax, a, b, _flags(ax, prec) | ax.ACC_TILE_128)
    assert np.array_equal(np.isfinite(c), np.isfinite(forced))
    fin = np.isfinite(c)
    assert fin.sum() == (m - 2) * (n - 1) and rel_fro(c[fin], forced[fin]) <= FP32_REL_FRO_TOL


def _direct_i8(ax, a, b, *args):
    import torch
    ax.accx_timing_enable(True)
    ax.accx_timing_read(reset=True)
    c = _run_i8(ax, a, b, *args)
    names = set(ax.accx_timing_read(reset=True))
    ax.accx_timing_enable(False)
    torch.cuda.synchronize()
    assert names == {"gemm_i8_direct"}, names
    return c


# at least three whole 64-element stages (the steady loop), with and without a
# tail; two K parts
I8_SHAPES = [(1100, 1157, 192), (1100, 1157, 257), (2048, 1800, 300), (129, 8100, 2100)]


@pytest.mark.parametrize("kind", ["one", "two", "three", "four"])
@pytest.mark.parametrize("m,n,k", I8_SHAPES)
def test_i32(ax, m, n, k, kind):
    a, b = _values(kind, (m, k), 9720 + m), _values(kind, (k, n), 9721 + n)
    ref = oracle.gemm(a, b)
    assert np.array_equal(_direct_i8(ax, a, b), ref)
    if k < 1000:
        for pad, offset in [((3, 1), (1, 3)), ((4, 8), (2, 0))]:
            assert np.array_equal(_direct_i8(ax, a, b, pad, offset), ref)


@pytest.mark.parametrize("m,n,k", [(1100, 1157, 300), (129, 8100, 2100), (130, 75, 4200)])
def test_i32_digit_count_changes_along_k(ax, m, n, k):
    # each 70-element stretch of K has another digit count, on one operand
    # only, on both, or neither, so that planes 1-3 of a stage's buffer fall
    # out of use and come back (130 x 75 x 4200: the smaller tile, K parts)
    g = synth.rng(SEED, 99)
    a, b = _values("one", (m, k), 9730), _values("one", (k, n), 9731)
    edge = np.array([127, -128, 128, -129, 32767, -32768, 32768, 8388607, -8388608, 8388608, 2147483647, -2147483648,
                     -1, 0, 1], np.int64).astype(np.int32)
    for s in range(0, k, 70):
        if (s // 70) % 4 in (1, 3):
            a[:, s:s + 70] = g.choice(edge, (m, min(70, k - s)))
        if (s // 70) % 4 in (2, 3):
            b[s:s + 70] = g.choice(edge, (min(70, k - s), n))
    assert np.array_equal(_direct_i8(ax, a, b), oracle.gemm(a, b))
