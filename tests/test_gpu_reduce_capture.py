"""Reductions on the null stream while a stream that synchronises with it is
being captured: a plain launch there, in any capture mode and at any number of
launches, and no part of the capture."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ax():
    import paper_1412_1127_amd as ax
    ax.acc_init(0, 0)
    yield ax
    ax.acc_shutdown()


@pytest.mark.parametrize("mode", [0, 1, 2])                  # global, thread local, relaxed
@pytest.mark.parametrize("n", [100, 100003, 5 * 2 ** 20])    # one workgroup, one launch, two launches
def test_null_stream_beside_a_capture(ax, mode, n):
    import torch
    hip = ctypes.CDLL("libamdhip64.so")
    x = np.arange(n, dtype=np.int32) % 17
    want = int(x.sum(dtype=np.int64)) + 5
    dx = torch.from_numpy(x).cuda()
    res = torch.zeros(2, dtype=torch.int32, device="cuda")
    need = ax.accx_reduce_vars_workspace_size(ax.ACC_INT32, n, [(ax.ACC_RED_SUM, 0), (ax.ACC_RED_MAX, 0)])
    work = torch.zeros(need, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    stream = ctypes.c_void_p()
    assert hip.hipStreamCreateWithFlags(ctypes.byref(stream), ctypes.c_uint(0)) == 0
    assert hip.hipStreamBeginCapture(stream, ctypes.c_int(mode)) == 0
    graph = ctypes.c_void_p()
    print("reduction beside a capture mode=%d n=%d" % (mode, n), flush=True)
    try:
        ax.accx_reduce_dev(ax.ACC_INT32, dx, n, [(ax.ACC_RED_SUM, 0)], [0], res, 0, work, need, stream=0)
        ax.accx_reduce_dev(ax.ACC_INT32, dx, n, [(ax.ACC_RED_SUM, 0), (ax.ACC_RED_MAX, 0)], [5, 0], res, 0, work, need,
                           stream=0)
    finally:
        ended = hip.hipStreamEndCapture(stream, ctypes.byref(graph))
        if ended == 0 and graph.value:
            hip.hipGraphDestroy(graph)
        hip.hipStreamDestroy(stream)
    torch.cuda.synchronize()
    assert ended == 0
    assert res.cpu().tolist() == [want, 16]
