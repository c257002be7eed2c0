"""A deposit recorded into a graph uses the scratch that earlier deposits left, also where it would
count its tiles row by row and has no room for the rows' counts yet."""
import numpy as np
import pytest

from oracle import grid as og
from paper_2008_10468_amd import qed
from test_gpu_grid import _deposit_mode, _grid, _particles

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("recorder", ("caller", "library"))
def test_recorded_without_rows(recorder):
    """Warmed on 129 x 128 x 64 cells (16,896 tiles: not row by row), recorded on 128 x 128 x 64
    (16,384 tiles: row by row); three replays with eager work between them.  Currents to 1e-10
    of the largest, as for the other deposits (double sums in another order)."""
    rng = np.random.default_rng(5)
    stream = torch.cuda.Stream()
    n = 300001
    with torch.cuda.stream(stream):
        gen = qed.Generator(precision=qed.QED_PREC_MIXED, capacity=(n, 16, 16), stream=stream.cuda_stream)
        big, sbig, keep = _grid(qed, gen.real, rng, 129, 128, 64)
        g, s, keep2 = _grid(qed, gen.real, rng, 128, 128, 64)
        gen.sp[0].upload(_particles(g, rng, n))
        _deposit_mode(qed, gen, "sorted")
        q = gen.sp[0].download()
        ref = og.deposit(g, q["x"], q["y"], q["z"], q["ux"], q["uy"], q["uz"], q["w"], -1.0)
        jbig = torch.zeros(3, 129 * 128 * 64, dtype=torch.float64, device="cuda")
        j = torch.zeros(3, 128 * 128 * 64, dtype=torch.float64, device="cuda")
        sp = gen.sp[0].struct()

        def deposit(grid, t):
            assert qed.qed_deposit(gen.ctx, grid, sp, -1.0, *[v.data_ptr() for v in t]) == qed.QED_OK
        deposit(sbig, jbig)
        stream.synchronize()
        if recorder == "caller":
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                deposit(s, j)
            replay = graph.replay
        else:
            assert qed.qed_graph_begin(gen.ctx) == qed.QED_OK
            deposit(s, j)
            st, handle = qed.qed_graph_end(gen.ctx)
            assert st == qed.QED_OK
            replay = lambda: qed.qed_graph_launch(gen.ctx, handle)   # noqa: E731
        for k in range(3):
            j.zero_()
            replay()
            stream.synchronize()
            for t, r in zip(j.cpu().numpy(), ref):
                assert np.abs(t - r).max() <= 1e-10 * np.abs(r).max()
            if k == 1:
                deposit(s, j)           # eager: takes the rows' counts
                deposit(sbig, jbig)
                stream.synchronize()
        if recorder == "library":
            qed.qed_graph_destroy(handle)
        gen.close()
