"""The correction of marked tiles from the float32 operands, over the probe's
list: few and many marked tiles, ragged sub-tiles, one and several K parts,
every probed tile of 128 x 128 and larger, against the oracle."""
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
    # terms of one sign: what the three products drop adds up (2.3e-5)
    h = 1.0 + g.integers(0, 16, shape) * 2.0 ** -7
    m = 2.0 ** -9 * (1.0 + g.integers(64, 128, shape) * 2.0 ** -7)
    l = 2.0 ** -18 * (1.0 + g.integers(16, 32, shape) * 2.0 ** -5)
    return (h + m + l).astype(np.float32)


@pytest.mark.parametrize("tile", ["128", "256", "256x128", "256w4"])
@pytest.mark.parametrize("m,n,k,rows", [(300, 400, 257, 300), (640, 900, 700, 130), (129, 257, 1, 129),
                                        (700, 300, 3000, 260)])
def test_marked_rows(ax, tile, m, n, k, rows):
    # the first `rows` rows of A are biased, the others hold one bf16 term per
    # element (three products are exact there): only tiles that touch the
    # first rows are marked
    import torch

    import paper_1412_1127_amd as pk
    g = synth.rng(SEED, 91)
    a = (g.integers(-128, 128, (m, k)) * 2.0 ** -7).astype(np.float32)
    a[:rows] = _biased(g, (rows, k))
    b = _biased(g, (k, n))
    fl = ax.ACC_KERNEL_TILED | ax.ACC_PREC_AUTO | pk.TILES[tile]
    ws = ax.accx_gemm_workspace_size(ax.ACC_FLOAT32, m, n, k, fl)
    off, cnt = ax.accx_gemm_probe_layout(m, n, k, fl)
    da, db = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    ref = oracle.gemm(a, b)
    first = None
    for rep in range(3):
        dc = torch.full((m, n), float("nan"), device="cuda")
        work = torch.randint(0, 255, (ws,), dtype=torch.uint8, device="cuda")
        print("correction tile=%s m=%d n=%d k=%d rep=%d" % (tile, m, n, k, rep), flush=True)
        ax.accx_gemm_dev(ax.ACC_FLOAT32, m, n, k, da, k, db, n, dc, n, fl, work, ws)
        torch.cuda.synchronize()
        c = dc.cpu().numpy()
        # (a tile that is biased in part is marked only if its samples are)
        h = 128 if tile == "128" else 256
        whole = rows if rows == m else rows // h * h
        assert rel_fro(c[:whole], ref[:whole]) <= FP32_REL_FRO_TOL
        assert rel_fro(c[rows:], ref[rows:]) <= FP32_REL_FRO_TOL
        first = c if first is None else first
        assert np.array_equal(c, first)   # the list's order does not show
        recs = ax.probe_records(work[off:off + cnt * 608].cpu().numpy().tobytes(), cnt)
        if k > 16:
            assert all(r.corrected for r in recs if max(r.rows) < rows)


@pytest.mark.parametrize("bad", [1, 700, 4096])
def test_open_tile_k_parts(ax, bad):
    # LEN = 4096 with the tile left open: `bad` biased rows, so one row of
    # tiles or all of them are marked; K parts per sub-tile follow from the
    # count.  Sampled rows against the oracle, the same bits on every run.
    import torch
    n = 4096
    g = synth.rng(SEED, 92)
    a = (g.integers(-128, 128, (n, n)) * 2.0 ** -7).astype(np.float32)
    a[:bad] = _biased(g, (bad, n))
    b = _biased(g, (n, n))
    da, db = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    rows = np.unique(np.concatenate([[0, bad - 1, bad // 2, n - 1], g.integers(0, n, 12)]))
    ref = oracle.gemm(np.ascontiguousarray(a[rows]), b)
    outs = []
    for rep in range(2):
        dc = torch.full((n, n), float("nan"), device="cuda")
        print("correction LEN=4096 bad=%d rep=%d" % (bad, rep), flush=True)
        ax.accx_matmul_dev(ax.ACC_FLOAT32, da, db, dc, n, 0)
        torch.cuda.synchronize()
        outs.append(dc)
    assert torch.equal(outs[0], outs[1])
    c = outs[0].cpu().numpy()[rows]
    assert np.isfinite(c).all()
    # rows of tiles that are biased throughout, or not at all
    keep = rows < bad // 256 * 256
    assert rel_fro(c[keep], ref[keep]) <= FP32_REL_FRO_TOL
    assert rel_fro(c[rows >= bad], ref[rows >= bad]) <= FP32_REL_FRO_TOL
