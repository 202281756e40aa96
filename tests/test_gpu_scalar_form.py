"""Which of its three launch forms the scalar layer takes where the measured costs lie far apart."""
import numpy as np
import pytest

from oracle import gcn
from paper_2511_09261_amd import inputs
from tests.parity import rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,rows,edges_per_row,form", [
    (16, 125, 2, "one_launch"),
    (4000, 3, 1, "one_launch"),   # staged: three launches of a workgroup per subgraph, 74 us against 33
    (12000, 3, 1, "one_launch"),
    (1, 5000, 3, "staged"),       # one workgroup: 66 us against 26
    (16, 5000, 5, "staged"),      # 96 us against 29
    (1, 20455, 15, "streams"),    # three rows too long for the staged form: 51 us, one workgroup 956
])
def test_the_form_follows_the_measured_costs(gco, P, rows, edges_per_row, form):
    rs = np.random.RandomState(P)
    n = P * rows
    base = rs.randint(0, P, edges_per_row * n) * rows
    g = inputs.from_edges(n, base + rs.randint(0, rows, base.size), base + rs.randint(0, rows, base.size))
    ctx = gco.Context(num_layers=1, dim=8, weight_sharing=True)
    ctx.upload_graph(n, g.rowptr, g.col, np.repeat(np.arange(P), rows).astype(np.int32), P)
    assert ctx.get_scalar_layer_form() == form
    ctx.destroy()


@pytest.mark.parametrize("edges", [2400, 2600, 2800, 6000])
def test_one_launch_holds_a_wavefronts_entries_or_streams_them(gco, edges):
    """The sixteen wavefronts of a subgraph keep up to 512 entries each in registers: a little below that, some
    on either side, and above; a transpose that differs.  fp32 sums of a few tens of terms against fp64."""
    rs = np.random.RandomState(edges)
    rows, P = 3000, 2
    base = rs.randint(0, P, edges * P) * rows
    g = inputs.from_edges(P * rows, base + rs.randint(0, rows, base.size), base + rs.randint(0, rows, base.size))
    part = np.repeat(np.arange(P), rows).astype(np.int32)
    E, Ws = inputs.init_params(g.n, part, P, 2, 8, 3)
    ctx = gco.Context(num_layers=2, dim=8, norm="mean")
    ctx.set_scalar_layer_form("one_launch")
    ctx.upload_graph(g.n, g.rowptr, g.col, part, P)
    ctx.set_params(E, Ws)
    spec = gcn.Spec(num_layers=2, norm="mean")
    lg = gcn.local_graph(g.n, g.rowptr, g.col, part, P, "mean")
    cache = gcn.forward(lg, E, Ws, spec)
    gE, gWs = gcn.backward(lg, cache, Ws, spec)
    dE, dWs = ctx.get_grads()
    assert rel(ctx.get_probs(), cache["p"]) <= 1e-5
    assert rel(dE, gE) <= 1e-5
    assert all(rel(d, w) <= 1e-5 for d, w in zip(dWs, gWs))
    ctx.destroy()
