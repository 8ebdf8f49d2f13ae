"""C sharing memory with an operand: the tiled path reads both operands before
it stores C, whichever way a shape is routed, so the result is that of the
operands as they were (small products and corrected tiles are otherwise run by
kernels that read the operands while C is written)."""
import numpy as np
import pytest

import oracle
import synth
from _util import FP32_REL_FRO_TOL, SEED, rel_fro

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ax():
    import paper_1412_1127_amd as ax
    ax.acc_init(0, 0)
    yield ax
    ax.acc_shutdown()


def _biased(g, shape):
    # terms of one sign: the probe marks every tile (2.3e-5 without the correction)
    h = 1.0 + g.integers(0, 16, shape) * 2.0 ** -7
    m = 2.0 ** -9 * (1.0 + g.integers(64, 128, shape) * 2.0 ** -7)
    l = 2.0 ** -18 * (1.0 + g.integers(16, 32, shape) * 2.0 ** -5)
    return (h + m + l).astype(np.float32)


def _check(c, a, b):
    ref = oracle.gemm(a, b)
    if a.dtype == np.int32:
        assert np.array_equal(c, ref)
    else:
        assert rel_fro(c, ref) <= FP32_REL_FRO_TOL


# (the forced tile corrects marked tiles from a list; 64 x 64 tiles and K parts
# at 200, 128 x 128 at 1500)
@pytest.mark.parametrize("n", [63, 200, 1500])
@pytest.mark.parametrize("kind", ["auto", "auto_marked", "full6", "auto_tile_128", "i32", "i32_full"])
@pytest.mark.parametrize("where", ["a", "b", "rows_into_a", "rows_into_b"])
def test_square(ax, n, kind, where):
    import torch
    if n == 1500 and where.startswith("rows"):
        n = 1499
    g = synth.rng(SEED, 95)
    t, flags = ax.ACC_FLOAT32, ax.ACC_KERNEL_TILED
    if kind.startswith("i32"):
        t = ax.ACC_INT32
        a, b = [synth.full_range_i32((n, n), SEED, 9400 + q) if kind == "i32_full" else
                synth.int_uniform_i32((n, n), -16, 16, SEED, 9400 + q) for q in range(2)]
    elif kind in ("auto_marked", "auto_tile_128"):
        a, b = _biased(g, (n, n)), _biased(g, (n, n))
        flags |= ax.ACC_TILE_128 if kind == "auto_tile_128" else 0
    else:
        a, b = synth.uniform_pm1_f32((n, n), SEED, 9400), synth.uniform_pm1_f32((n, n), SEED, 9401)
        flags |= ax.ACC_PREC_FULL6 if kind == "full6" else 0
    shift = 37 * n if where.startswith("rows") else 0   # C starts 37 rows into the operand
    buf = [torch.zeros(2 * n * n, dtype=torch.from_numpy(a).dtype, device="cuda") for _ in range(2)]
    buf[0][:n * n] = torch.from_numpy(a.reshape(-1)).cuda()
    buf[1][:n * n] = torch.from_numpy(b.reshape(-1)).cuda()
    c = buf[0 if where.endswith("a") else 1][shift:shift + n * n]
    print("overlap n=%d kind=%s where=%s" % (n, kind, where), flush=True)
    ax.accx_matmul_dev(t, buf[0], buf[1], c, n, flags)
    torch.cuda.synchronize()
    _check(c.cpu().numpy().reshape(n, n), a, b)


@pytest.mark.parametrize("kind", ["auto", "i32"])
def test_c_in_the_padding_of_a(ax, kind):
    # the spans overlap, the elements do not
    import torch
    m, n, k = 130, 70, 90
    if kind == "i32":
        a, b = synth.int_uniform_i32((m, k), -16, 16, SEED, 9410), synth.int_uniform_i32((k, n), -16, 16, SEED, 9411)
    else:
        a, b = synth.uniform_pm1_f32((m, k), SEED, 9410), synth.uniform_pm1_f32((k, n), SEED, 9411)
    ac = torch.zeros((m, k + n), dtype=torch.from_numpy(a).dtype, device="cuda")
    ac[:, :k] = torch.from_numpy(a).cuda()
    db = torch.from_numpy(b).cuda()
    print("overlap C in the padding of A, %s" % kind, flush=True)
    ax.accx_gemm_dev(ax.ACC_INT32 if kind == "i32" else ax.ACC_FLOAT32, m, n, k, ac, k + n, db, n,
                     ac[:, k:].data_ptr(), k + n, ax.ACC_KERNEL_TILED)
    torch.cuda.synchronize()
    out = ac.cpu().numpy()
    assert np.array_equal(out[:, :k], a)
    _check(out[:, k:], a, b)


@pytest.mark.parametrize("kind", ["uniform", "marked"])
@pytest.mark.parametrize("m,n,k", [(70, 50, 2049), (130, 200, 1500), (100, 1100, 300)])
def test_rows_too_long_for_the_direct_path(ax, m, n, k, kind):
    # rows further apart than the direct kernels' offsets reach: packed, on the
    # tile and with the split K of the three-product call, so that the
    # two agree bit for bit on unmarked tiles; marked ones are corrected
    import torch
    lda = (1 << 19) + 8
    g = synth.rng(SEED, 97)
    if kind == "marked":
        a, b = _biased(g, (m, k)), _biased(g, (k, n))
    else:
        a, b = synth.uniform_pm1_f32((m, k), SEED, 9420), synth.uniform_pm1_f32((k, n), SEED, 9421)
    buf = torch.zeros((m - 1) * lda + k, device="cuda")
    buf.as_strided((m, k), (lda, 1)).copy_(torch.from_numpy(a))
    db = torch.from_numpy(b).cuda()
    fl = ax.ACC_KERNEL_TILED | ax.ACC_PREC_AUTO
    ws = ax.accx_gemm_workspace_size(ax.ACC_FLOAT32, m, n, k, fl)
    off, cnt = ax.accx_gemm_probe_layout(m, n, k, fl)
    work = torch.full((ws,), 0xFF, dtype=torch.uint8, device="cuda")
    out = []
    for flags in (fl, ax.ACC_KERNEL_TILED | ax.ACC_PREC_CHEAP3):
        dc = torch.full((m, n), float("nan"), device="cuda")
        print("long rows m=%d n=%d k=%d %s flags=%#x" % (m, n, k, kind, flags), flush=True)
        ax.accx_gemm_dev(ax.ACC_FLOAT32, m, n, k, buf, lda, db, n, dc, n, flags, work if flags == fl else None,
                         ws if flags == fl else 0)
        torch.cuda.synchronize()
        out.append(dc.cpu().numpy())
    recs = ax.probe_records(work[off:off + cnt * 608].cpu().numpy().tobytes(), cnt)
    assert rel_fro(out[0], oracle.gemm(a, b)) <= FP32_REL_FRO_TOL
    edge = next(e for e in (64, 128) if -(-m // e) * -(-n // e) == cnt)
    nt = -(-n // edge)
    if kind == "marked":
        assert all(r.corrected for r in recs)
    else:
        # (a sampled error of this kind of values is rarely above the threshold)
        assert sum(r.corrected for r in recs) <= cnt // 4
    for q, r in enumerate(recs):
        at = np.s_[q // nt * edge:(q // nt + 1) * edge, q % nt * edge:(q % nt + 1) * edge]
        assert np.array_equal(out[0][at], out[1][at]) == (not r.corrected)
