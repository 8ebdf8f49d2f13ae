"""One-launch reductions of every element type against the two launches that a
capture records, bit for bit, and many of them in flight on two streams, each
with a workspace of its own."""
import numpy as np
import pytest

import oracle
import synth
from _util import SEED

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ax():
    import paper_1412_1127_amd as ax
    ax.acc_init(0, 0)
    yield ax
    ax.acc_shutdown()


# one workgroup, one arrival word, two levels, beyond a plain sum's one launch
@pytest.mark.parametrize("n", [100, 100003, 300 * 8192 + 5, 600 * 8192 + 1])
@pytest.mark.parametrize("which", ["sum", "four"])
@pytest.mark.parametrize("kind", ["i32", "i64"])
def test_integers_equal_captured(ax, kind, which, n):
    import torch
    t, dt = (ax.ACC_INT32, torch.int32) if kind == "i32" else (ax.ACC_INT64, torch.int64)
    x = synth.full_range_i32((n,), SEED, 9800)
    if kind == "i64":
        x = x.astype(np.int64) * 0x100000001 + 12345
    s, mx, mn = ax.ACC_RED_SUM, ax.ACC_RED_MAX, ax.ACC_RED_MIN
    vars_ = [(s, 0)] if which == "sum" else [(s, 1), (mx, 0), (mn, 1), (s, 0)]
    init = [3, -7, 11, -13][:len(vars_)]
    dx = torch.from_numpy(x).cuda()
    need = ax.accx_reduce_vars_workspace_size(t, n, vars_)
    work = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
    res = torch.zeros(len(vars_), dtype=dt, device="cuda")
    print("reduce %s %s n=%d" % (kind, which, n), flush=True)
    ax.accx_reduce_dev(t, dx, n, vars_, init, res, 0, work, need)
    torch.cuda.synchronize()
    eager = res.cpu().numpy().copy()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ax.accx_reduce_dev(t, dx, n, vars_, init, res, 0, work, need, stream=torch.cuda.current_stream().cuda_stream)
    for fill in (255, 0, 3):
        work.fill_(fill)
        res.fill_(55)
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(res.cpu().numpy(), eager)
    ops = {s: "sum", mx: "max", mn: "min"}
    want = [oracle.reduce(x, ops[op], i, square=bool(sq)) for (op, sq), i in zip(vars_, init)]
    assert [int(v) for v in eager] == [int(v) for v in want]


def test_two_streams_in_flight(ax):
    import torch
    sizes = [100003, 300 * 8192 + 5, 700 * 8192 + 3]
    vars_ = [(ax.ACC_RED_SUM, 0), (ax.ACC_RED_SUM, 1)]
    x = torch.from_numpy(synth.uniform01_f32(max(sizes), SEED, 9810)).cuda()
    need = ax.accx_reduce_vars_workspace_size(ax.ACC_FLOAT32, max(sizes), vars_)
    want = {}
    for n in sizes:
        r = torch.empty(2, device="cuda")
        ax.accx_reduce_dev(ax.ACC_FLOAT32, x, n, vars_, [0.0, 0.0], r)
        torch.cuda.synchronize()
        want[n] = r.clone()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    works = [torch.full((need,), 0xA5 + k, dtype=torch.uint8, device="cuda") for k in range(2)]
    res = [torch.zeros((60, 2), device="cuda") for _ in range(2)]
    torch.cuda.synchronize()
    print("reductions on two streams", flush=True)
    for k in range(60):
        for q in range(2):
            n = sizes[(k + q) % 3]
            # every other call on the library's workspace of that stream
            w, b = (works[q], need) if k % 2 else (None, 0)
            ax.accx_reduce_dev(ax.ACC_FLOAT32, x, n, vars_, [0.0, 0.0], res[q][k], 0, w, b, stream=streams[q])
    torch.cuda.synchronize()
    for q in range(2):
        for k in range(60):
            assert torch.equal(res[q][k], want[sizes[(k + q) % 3]]), (q, k)
