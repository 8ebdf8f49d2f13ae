"""Batched matmuls straight from the float32 operands: every tile the size
policy picks at the edges of tiles and K stages, bitwise against the
standalone call on the same tile, and operands that some item of the batch
overwrites."""
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


def _inputs(n, k):
    return (synth.uniform_pm1_f32((n, n), SEED, 7000 + 2 * k), synth.uniform_pm1_f32((n, n), SEED, 7001 + 2 * k))


@pytest.mark.parametrize("auto", [False, True])
@pytest.mark.parametrize("lens", [[1, 2, 15, 16, 17, 31, 32, 33, 47], [63, 64, 65, 95, 97, 127, 128, 129],
                                  [255, 256, 257, 383, 384, 385], [511, 512, 513, 640, 700]])
def test_tile_and_stage_edges(ax, lens, auto):
    import torch
    mats = []
    for k, n in enumerate(lens):
        a, b = _inputs(n, k)
        mats.append((n, a, b, torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda(),
                     torch.full((n, n), float("nan"), device="cuda")))
    print("batch lens=%s auto=%d" % (lens, auto), flush=True)
    h = ax.accx_batch_create([ax.batch_matmul(da, db, dc, n) for n, _a, _b, da, db, dc in mats],
                             ax.ACC_BATCH_PREC_AUTO if auto else 0)
    ax.accx_batch_launch(h)
    torch.cuda.synchronize()
    prec = ax.ACC_PREC_AUTO if auto else ax.ACC_PREC_FULL6
    for n, a, b, da, db, dc in mats:
        c = dc.cpu().numpy()
        assert rel_fro(c, oracle.matmul_f32(a, b)) <= FP32_REL_FRO_TOL, n
        # the policy's tile, standalone and unsplit (a workspace without the
        # split area): the same bits on one of them
        w = 2 * ax.accx_packed_size(ax.ACC_FLOAT32, n, n, 3)
        if auto:
            off, _ = ax.accx_probe_layout(n, ax.ACC_KERNEL_TILED | prec)
            _, cnt = ax.accx_probe_layout(n, ax.ACC_KERNEL_TILED | prec | ax.ACC_TILE_64)
            w = off + cnt * 608
        solos = []
        for tile in (ax.ACC_TILE_64, ax.ACC_TILE_128, ax.ACC_TILE_256x128):
            flags = ax.ACC_KERNEL_TILED | prec | tile
            solo = torch.empty_like(dc)
            work = torch.empty(w, dtype=torch.uint8, device="cuda")
            ax.accx_matmul_dev(ax.ACC_FLOAT32, da, db, solo, n, flags, work, w)
            torch.cuda.synchronize()
            solos.append(np.array_equal(c, solo.cpu().numpy()))
        assert any(solos), n
    ax.accx_batch_destroy(h)


def test_operands_that_the_batch_overwrites(ax):
    # in place (c is a, c is b), one item's result inside another's operand,
    # and a reduction's result inside an operand: every matmul sees its
    # operands as they are when the batch is launched, on every launch
    import torch
    n = 96
    x = [torch.from_numpy(synth.uniform_pm1_f32((n, n), SEED, 7100 + k)).cuda() for k in range(6)]
    keep = [v.clone() for v in x]
    r = torch.ones(1000, device="cuda")
    items = [ax.batch_matmul(x[0], x[1], x[0], n),   # c is a
             ax.batch_matmul(x[2], x[3], x[3], n),   # c is b
             ax.batch_matmul(x[3], x[4], x[5], n),   # reads the item above's result array
             ax.batch_reduce(r, 1000, x[4][n - 1, n - 1:])]
    print("batch with overwritten operands", flush=True)
    h = ax.accx_batch_create(items, ax.ACC_BATCH_PREC_AUTO)
    for rep in range(3):
        for v, k in zip(x, keep):
            v.copy_(k)
        torch.cuda.synchronize()
        ax.accx_batch_launch(h)
        torch.cuda.synchronize()
        a = [k.cpu().numpy() for k in keep]
        for c, (p, q) in ((x[0], (0, 1)), (x[3], (2, 3)), (x[5], (3, 4))):
            assert rel_fro(c.cpu().numpy(), oracle.matmul_f32(a[p], a[q])) <= FP32_REL_FRO_TOL, (rep, p, q)
        assert float(x[4][n - 1, n - 1].item()) == 1000.0
    ax.accx_batch_destroy(h)
