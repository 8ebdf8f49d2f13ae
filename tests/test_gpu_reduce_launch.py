"""Reductions whose last arriving workgroup folds the partials (one launch)
against the two-launch form that a capture records: both add the same
partials in the same order, so they agree bit for bit, whatever the workspace
held before.  The sizes give one workgroup, two, three, the largest number
that arrives at one word (for either element type) and one more, the largest
that takes one launch for a plain sum and one more, and a full grid, with
ragged ends."""
import numpy as np
import pytest

import oracle
import synth
from _util import SEED

pytestmark = pytest.mark.gpu

SIZES = [1, 8192, 8197, 16389, 100003, 32 * 8192 + 1, 64 * 8192 + 3, 64 * 8192 + 4, 512 * 8192, 512 * 8192 + 4,
         768 * 8192 + 8195]


@pytest.fixture(scope="module")
def ax():
    import paper_1412_1127_amd as ax
    ax.acc_init(0, 0)
    yield ax
    ax.acc_shutdown()


def _vars(ax, which):
    s, m, n = ax.ACC_RED_SUM, ax.ACC_RED_MAX, ax.ACC_RED_MIN
    return {"sum": [(s, 0)], "sumsq": [(s, 0), (s, 1)], "four": [(s, 1), (m, 0), (n, 1), (s, 0)]}[which]


@pytest.mark.parametrize("which", ["sum", "sumsq", "four"])
@pytest.mark.parametrize("n", SIZES)
def test_one_launch_equals_captured(ax, n, which):
    import torch
    vars_ = _vars(ax, which)
    init = [0.5, -0.25, 2.0, 0.125][:len(vars_)]
    for t, dt, x in [(ax.ACC_FLOAT32, torch.float32, synth.uniform01_f32(n, SEED, 760)),
                     (ax.ACC_FLOAT64, torch.float64, synth.uniform_pm1_f64(n, SEED, 761))]:
        dx = torch.from_numpy(x).cuda()
        need = ax.accx_reduce_vars_workspace_size(t, n, vars_)
        work = torch.zeros(need, dtype=torch.uint8, device="cuda")
        res = torch.zeros(len(vars_), dtype=dt, device="cuda")
        print("one launch n=%d vars=%s type=%d" % (n, which, t), flush=True)

        def run(fill):
            work.fill_(fill)
            res.fill_(77)
            ax.accx_reduce_dev(t, dx, n, vars_, init, res, 0, work, need)
            torch.cuda.synchronize()
            return res.cpu().numpy().tobytes()

        eager = [run(f) for f in (0, 1, 255)]
        ax.accx_reduce_dev(t, dx, n, vars_, init, res, 0, work, need)  # on what the last one left
        torch.cuda.synchronize()
        eager.append(res.cpu().numpy().tobytes())
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            ax.accx_reduce_dev(t, dx, n, vars_, init, res, 0, work, need,
                               stream=torch.cuda.current_stream().cuda_stream)
        for fill in (255, 0, 3):
            work.fill_(fill)
            res.fill_(55)
            graph.replay()
            torch.cuda.synchronize()
            eager.append(res.cpu().numpy().tobytes())
        assert all(e == eager[0] for e in eager)
        got = np.frombuffer(eager[0], dtype=x.dtype)
        for v, (op, sq) in enumerate(vars_):
            want = oracle.reduce(x, {ax.ACC_RED_SUM: "sum", ax.ACC_RED_MAX: "max", ax.ACC_RED_MIN: "min"}[op],
                                 init[v], square=bool(sq))
            scale = max(abs(want), float(np.sqrt(n)))  # sums of values around zero cancel
            assert abs(float(got[v]) - want) <= (1e-5 if t == ax.ACC_FLOAT32 else 1e-12) * scale
