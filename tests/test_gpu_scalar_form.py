"""Which of its three launch forms the scalar layer takes where the measured costs lie far apart."""
import numpy as np
import pytest

from paper_2511_09261_amd import inputs

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
