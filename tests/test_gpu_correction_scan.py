"""Marked tiles of a direct product in more than one round of tiles: corrected
by a launch that finds them in the probe's records.  Few, many, all and no
marked tiles, ragged ones, one and several K parts, a workspace of any
contents, against the oracle.  (More than one round: sizes for 256 compute
units.)"""
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


def _biased(g, shape):
    # terms of one sign: what the three products drop adds up (2.3e-5)
    h = 1.0 + g.integers(0, 16, shape) * 2.0 ** -7
    m = 2.0 ** -9 * (1.0 + g.integers(64, 128, shape) * 2.0 ** -7)
    l = 2.0 ** -18 * (1.0 + g.integers(16, 32, shape) * 2.0 ** -5)
    return (h + m + l).astype(np.float32)


# 289, 576, 288 and 640 records (the most there are); rows of A that are
# biased (a multiple of 128, or all), the others hold one bf16 term per
# element, for which three products are exact
@pytest.mark.parametrize("m,n,k,rows", [(2060, 2150, 600, 2060), (2060, 2150, 800, 128), (2060, 2150, 800, 1024),
                                        (2060, 2150, 600, 0), (2950, 2950, 520, 2950), (9100, 500, 1100, 256),
                                        (2550, 4090, 512, 2550), (2060, 2150, 511, 2060), (2950, 2950, 40, 384),
                                        (2200, 2200, 1, 0)])
def test_marked_tiles(ax, m, n, k, rows):
    import torch
    g = synth.rng(SEED, 96)
    a = (g.integers(-128, 128, (m, k)) * 2.0 ** -7).astype(np.float32)
    a[:rows] = _biased(g, (rows, k))
    b = _biased(g, (k, n))
    fl = ax.ACC_KERNEL_TILED | ax.ACC_PREC_AUTO
    ws = ax.accx_gemm_workspace_size(ax.ACC_FLOAT32, m, n, k, fl)
    off, cnt = ax.accx_gemm_probe_layout(m, n, k, fl)
    assert cnt == -(-m // 128) * -(-n // 128) > 256
    da, db = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    ref = oracle.gemm(a, b)
    first = None
    for fill in (0x00, 0xFF, 0x5A):
        dc = torch.full((m, n), float("nan"), device="cuda")
        work = torch.full((ws,), fill, dtype=torch.uint8, device="cuda")
        print("scan m=%d n=%d k=%d rows=%d fill=%#x" % (m, n, k, rows, fill), flush=True)
        ax.accx_timing_enable(True)
        ax.accx_timing_read(reset=True)
        ax.accx_gemm_dev(ax.ACC_FLOAT32, m, n, k, da, k, db, n, dc, n, fl, work, ws)
        torch.cuda.synchronize()
        names = set(ax.accx_timing_read(reset=True))
        ax.accx_timing_enable(False)
        # (short loops: each marked tile by the workgroup that found it)
        assert names == {"gemm_direct_auto"} | ({"gemm_bf16x3_corr"} if k >= 512 else set()), names
        c = dc.cpu().numpy()
        assert rel_fro(c[:rows], ref[:rows]) <= FP32_REL_FRO_TOL
        assert rel_fro(c[rows:], ref[rows:]) <= FP32_REL_FRO_TOL
        first = c if first is None else first
        assert np.array_equal(c, first)
        recs = ax.probe_records(work[off:off + cnt * 608].cpu().numpy().tobytes(), cnt)
        if k > 16:
            assert all(r.corrected == (1 if max(r.rows) < rows else 0) for r in recs)
