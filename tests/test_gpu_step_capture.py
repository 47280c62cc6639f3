"""Steps whose lists fit a kernel argument (3 KB) can be captured in a graph: at sizes just inside that, for query tiles that
are cut (one long request, with few and with many partials) and for whole ones (many short requests, few and many heads), every replay gives the eager result."""
import numpy as np
import pytest
import torch

from paper_2605_04450_amd import binding as B
from paper_2605_04450_amd import device as Hn
from tests.test_gpu_hstu import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,new", [(256, [32] * 31), (128, [20] * 35), (512, [5] * 24), (256, [60, 1300]), (64, [2300])])
def test_replays_equal_the_eager_step(d, new):
    c = Case(43, 2, d, d // 64, 64, True, 300, 16, 300.0, 256)
    reqs, pts, ts, x = c.inputs([0] * len(new), new)
    want = c.run_gpu(reqs, pts, ts, x)  # also makes room for the lists
    xd = torch.from_numpy(x).to(Hn.DEV).to(Hn.torch_dtype(c.elem))
    ptd, tsd, out = torch.from_numpy(pts).to(Hn.DEV), torch.from_numpy(ts).to(Hn.DEV), torch.empty_like(xd)
    torch.cuda.synchronize()
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=stream):
        assert B.hstu_step(c.pool.h, c.model.h, reqs, ptd, xd, tsd, out) == B.OK, B.last_error()
    for _ in range(3):
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.float().cpu().numpy(), want)
        assert np.array_equal(c.run_gpu(reqs, pts, ts, x), want)  # eager work between the replays
    c.close()
