"""The tile policy of a batch: 256 x 128 tiles where they fill the persistent
workgroups, 128 x 128 where they would leave some idle; and the results of
both, ragged tiles included, bit for bit those of the standalone calls on
that tile.  (Counts for 256 compute units.)"""
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
        pytest.skip("counts for 256 compute units")
    ax.acc_init(0, 0)
    yield ax
    ax.acc_shutdown()


def _tiles(lens, bm, bn):
    return sum(-(-n // bm) * -(-n // bn) for n in lens)


@pytest.mark.parametrize("lens,auto,wide", [
    ([2048], True, False), ([2048] * 2, True, False), ([2048] * 3, True, False), ([2048] * 4, True, True),
    ([1024] * 8, True, False), ([1024] * 16, True, True), ([2048] * 4, False, False), ([3584], True, True),
    ([700] * 21 + [64] * 40, True, False), ([700] * 22 + [64] * 40, True, True)])
@pytest.mark.parametrize("tuned", [False, True])
def test_tile_count(ax, lens, auto, wide, tuned):
    import torch
    total = sum(n * n for n in lens)
    a, b = torch.rand(total, device="cuda"), torch.rand(total, device="cuda")
    c = torch.empty(total, device="cuda")
    items, o = [], 0
    for n in lens:
        items.append(ax.batch_matmul(a[o:], b[o:], c[o:], n))
        o += n * n
    print("batch %d x %d auto=%d tuned=%d" % (len(lens), lens[0], auto, tuned), flush=True)
    h = ax.accx_batch_create(items, (ax.ACC_BATCH_PREC_AUTO if auto else 0) | (ax.ACC_BATCH_AUTOTUNE if tuned else 0))
    info = ax.accx_batch_info(h)
    ax.accx_batch_destroy(h)
    th = info["tile_threshold"]
    big, small = [n for n in lens if n >= th], [n for n in lens if n < th]
    assert info["tiles"] == _tiles(big, 256 if wide else 128, 128) + _tiles(small, 64, 64), info


@pytest.mark.parametrize("count", [4, 24])
def test_results_on_both(ax, count):
    # 24 matmuls: 396 tiles of 256 x 128 for the LENs that they cover at less
    # padding (700, 760), 128 x 128 for the others; 4: 128 x 128 for all.  Each
    # bit for bit as the standalone call with that tile forced, run unsplit
    import torch
    lens = [700, 760, 513, 640] + [700] * (count - 4)
    mats = []
    for k, n in enumerate(lens):
        a = synth.uniform_pm1_f32((n, n), SEED, 9600 + 2 * (k % 4))
        b = synth.uniform_pm1_f32((n, n), SEED, 9601 + 2 * (k % 4))
        mats.append((n, a, b, torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda(),
                     torch.full((n, n), float("nan"), device="cuda")))
    print("batch results %d matmuls" % count, flush=True)
    h = ax.accx_batch_create([ax.batch_matmul(da, db, dc, n) for n, _a, _b, da, db, dc in mats], ax.ACC_BATCH_PREC_AUTO)
    ax.accx_batch_launch(h)
    torch.cuda.synchronize()
    for n, a, b, da, db, dc in mats[:5]:
        flags = ax.ACC_KERNEL_TILED | ax.ACC_PREC_AUTO
        flags |= ax.ACC_TILE_256x128 if count == 24 and n in (700, 760) else ax.ACC_TILE_128
        c = dc.cpu().numpy()
        assert rel_fro(c, oracle.matmul_f32(a, b)) <= FP32_REL_FRO_TOL, n
        off, _ = ax.accx_probe_layout(n, flags)
        _, cnt = ax.accx_probe_layout(n, ax.ACC_KERNEL_TILED | ax.ACC_PREC_AUTO | ax.ACC_TILE_64)
        w = off + cnt * 608   # no room for split K
        work = torch.empty(w, dtype=torch.uint8, device="cuda")
        solo = torch.empty_like(dc)
        ax.accx_matmul_dev(ax.ACC_FLOAT32, da, db, solo, n, flags, work, w)
        torch.cuda.synchronize()
        assert np.array_equal(c, solo.cpu().numpy()), n
    ax.accx_batch_destroy(h)
