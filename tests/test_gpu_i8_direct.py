"""The int32 nest straight from its operands: bit-exact at the edges of tiles,
K stages, groups and parts, for every digit count, values whose digit count
changes along K, and rows of any alignment; and packing from such rows."""
import numpy as np
import pytest

import oracle
import synth
from _util import SEED

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (63, 65, 63), (64, 64, 64), (65, 63, 65), (33, 100, 127), (100, 33, 193), (128, 130, 257),
          (200, 72, 1000), (1030, 1100, 40), (1100, 1157, 65), (70, 50, 2049), (256, 256, 4100), (1300, 1211, 700),
          (130, 1, 3000), (1, 200, 2500)]


@pytest.fixture(scope="module")
def ax():
    import paper_1412_1127_amd as ax
    ax.acc_init(0, 0)
    yield ax
    ax.acc_shutdown()


def _values(kind, shape, stream):
    if kind == "one":
        return synth.int_uniform_i32(shape, -128, 127, SEED, stream)
    if kind == "two":
        return synth.int_uniform_i32(shape, -32768, 32767, SEED, stream)
    if kind == "three":
        return synth.int_uniform_i32(shape, -8388608, 8388607, SEED, stream)
    return synth.full_range_i32(shape, SEED, stream)


def _run(ax, a, b, pad=(0, 0), offset=(0, 0)):
    import torch
    m, k = a.shape
    n = b.shape[1]

    def put(x, p, o):
        buf = np.full(o + x.shape[0] * (x.shape[1] + p) + 4, 0x7fffffff, np.int32)
        buf[o:o + x.shape[0] * (x.shape[1] + p)].reshape(x.shape[0], -1)[:, :x.shape[1]] = x
        return torch.from_numpy(buf).cuda()

    da, db = put(a, pad[0], offset[0]), put(b, pad[1], offset[1])
    dc = torch.full((m, n + 1), 77, dtype=torch.int32, device="cuda")
    print("i8 m=%d n=%d k=%d pad=%s offset=%s" % (m, n, k, pad, offset), flush=True)
    ax.accx_gemm_dev(ax.ACC_INT32, m, n, k, da.data_ptr() + 4 * offset[0], max(1, k + pad[0]),
                     db.data_ptr() + 4 * offset[1], n + pad[1], dc, n + 1, ax.ACC_KERNEL_TILED)
    torch.cuda.synchronize()
    c = dc.cpu().numpy()
    assert (c[:, n] == 77).all(), "C padding written"
    return c[:, :n]


@pytest.mark.parametrize("kind", ["one", "two", "three", "four"])
@pytest.mark.parametrize("m,n,k", SHAPES)
def test_bit_exact_at_edges(ax, m, n, k, kind):
    a, b = _values(kind, (m, k), 9000 + m), _values(kind, (k, n), 9100 + n)
    ref = oracle.gemm(a, b)
    assert np.array_equal(_run(ax, a, b), ref)
    for pad, offset in [((3, 1), (1, 3)), ((4, 8), (2, 0))]:
        assert np.array_equal(_run(ax, a, b, pad, offset), ref)


@pytest.mark.parametrize("k", [200, 1000, 4200])
def test_digit_count_changes_along_k(ax, k):
    # each 50-element stretch of K has another digit count, on one operand
    # only, on both, or neither; the extremes of every digit among the values
    m, n = 130, 75
    g = synth.rng(SEED, 93)
    a, b = _values("one", (m, k), 9200), _values("one", (k, n), 9201)
    edge = np.array([127, -128, 128, -129, 32767, -32768, 32768, 8388607, -8388608, 8388608, 2147483647, -2147483648,
                     -1, 0, 1], np.int64).astype(np.int32)
    for s in range(0, k, 50):
        if (s // 50) % 4 in (1, 3):
            a[:, s:s + 50] = g.choice(edge, (m, min(50, k - s)))
        if (s // 50) % 4 in (2, 3):
            b[s:s + 50] = g.choice(edge, (min(50, k - s), n))
    assert np.array_equal(_run(ax, a, b), oracle.gemm(a, b))


@pytest.mark.parametrize("prec", ["full6", "i32"])
def test_packed_path_on_unaligned_rows(ax, prec):
    # a size the packed path takes, on rows that start at any 4-byte address
    import torch
    m, n, k = 2300, 2400, 133
    if prec == "i32":
        a, b = _values("two", (m, k), 9300), _values("two", (k, n), 9301)
        assert np.array_equal(_run(ax, a, b, (1, 3), (1, 2)), oracle.gemm(a, b))
        return
    a = synth.uniform_pm1_f32((m, k), SEED, 9300)
    b = synth.uniform_pm1_f32((k, n), SEED, 9301)
    outs = []
    for pad, off in ((0, 0), (1, 1), (2, 3)):
        buf = torch.full((off + m * (k + pad) + 4,), float("nan"), device="cuda")
        va = buf[off:off + m * (k + pad)].view(m, k + pad)
        va[:, :k] = torch.from_numpy(a).cuda()
        bufb = torch.full((off + k * (n + pad) + 4,), float("nan"), device="cuda")
        vb = bufb[off:off + k * (n + pad)].view(k, n + pad)
        vb[:, :n] = torch.from_numpy(b).cuda()
        c = torch.empty((m, n), device="cuda")
        print("packed rows pad=%d offset=%d" % (pad, off), flush=True)
        ax.accx_gemm_dev(ax.ACC_FLOAT32, m, n, k, va.data_ptr(), k + pad, vb.data_ptr(), n + pad, c, n,
                         ax.ACC_KERNEL_TILED | ax.ACC_PREC_FULL6)
        torch.cuda.synchronize()
        outs.append(c)
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    ref = oracle.gemm(a, b)
    assert np.linalg.norm(outs[0].cpu().numpy() - ref) <= 1e-5 * np.linalg.norm(ref)
